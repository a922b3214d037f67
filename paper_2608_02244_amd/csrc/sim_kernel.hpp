// Batched evaluation of the token-step scheduling model: one wavefront per
// instance.
//
// Model (Section 2): job i needs len_i = prompt_i + output_i steps; a job
// started at step s is active on s .. s+len-1; at most B jobs per step; the
// fairness constraint eq. (1) bounds the progress spread of co-running jobs by
// alpha; a KV budget M_kv bounds the summed reservations of co-running jobs.
// Policies: FCFS / SJF (Section 2.1 baselines), LJF (Algorithm 1) and ISJL
// (Algorithms 2 and 3 on the released queue, Section 3.5).  Costs: Section 5.
//
// The kernel is event driven.  Between two events (a completion, a release, a
// delayed plan start, or the step at which A_max(t) crosses alpha while Phase
// TWO waits on the KV budget) the active set is fixed and every active job
// advances one token per step, so the per-step terms of Section 5 are
// arithmetic series summed in closed form:
//   max r over [t, t+D): m_t = t - min_s + 1, sum = D m_t + D(D-1)/2
//   E per step  = sum_S (m_t - r_i) = sum_s - |S| min_s       (constant)
//   extent      = max_s - min_s                               (constant)
//   sum_S r     = |S| (t+1) - sum_s                            (largest at t+D-1)
// Decisions are taken only at events; the step-by-step definition gives the
// same decisions at the steps in between because nothing they depend on
// changes there.  (With the prompt prefilled at admission the largest
// footprint is t + max(prompt_j - start_j) + 1 and E per step is
// |S| G - sum_S (prompt_j - start_j), both constant between events.)
//
// Per-wave state:
//   LDS   W[r]     jobs in the policy's priority order, packed (len << 12 | id)
//         QN[r]    next job in the same ISJL plan queue (uint16, ISJL)
//         STG[j]   gather buffer of the first queued ranks (uint16, not FCFS)
//         PEND[i]  released ranks on their way into the bitmap, and up to 64
//                  slots or completions that a sweep packs (aliases STG; FCFS
//                  has it, 64 words, with 2 or more slots per lane or the prompt
//                  prefilled, and its other kernels never touch it)
//   The drain sweep sorts the active slots in registers; up to 64 of them are
//   first packed into one register through the gather buffer.
//   VGPR  K worker slots per lane: worker w lives in slot w/64 of lane w%64
//         (start, end, ISJL plan-queue head|tail); a bitmap of queued jobs over
//         ranks (bit r%32 of word r/2048 in lane (r/32)%64).
//   SGPR  time, counters, cost accumulators.
#pragma once
#include <type_traits>

#include "sim_common.hpp"
#include "regsort.hpp"
#include "wave.hpp"

namespace fs {

constexpr int POL_FCFS = FSCHED_FCFS, POL_LJF = FSCHED_LJF, POL_ISJL = FSCHED_ISJL,
              POL_SJF = FSCHED_SJF;
constexpr int IDLE = 0x7FFFFFFF;
constexpr uint32_t QNONE = 0xFFFFu;
constexpr uint32_t LMASK = 0xFFFFFu;

__device__ __forceinline__ int plen(uint32_t w) { return (int)(w >> 12); }
__device__ __forceinline__ int pid(uint32_t w) { return (int)(w & 0xFFFu); }

// Release order of jobs whose arrivals are not sorted by index: RK[i] holds the
// rank of job i on entry and the rank of the i-th released job afterwards (n
// entries, arrivals below 2^20).  Every load of the row has returned before the
// sort ends, so it is rewritten in place.
template <int KS>
__device__ inline void release_order(const int32_t* A, uint16_t* RK, int n, int lane) {
  uint32_t key[KS];
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    const int i = k * WAVE + lane;
    key[k] = i < n ? ((uint32_t)A[i] << 12) | RK[i] : 0xFFFFFFFFu;
  }
  reg_sort_keys<KS, true>(key, lane);
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    const int i = lane * KS + k;
    if (i < n) RK[i] = (uint16_t)(key[k] & 0xFFFu);
  }
}

__device__ inline void write_marker(fsched_metrics* out, int64_t* out_T, int64_t inst,
                                    int64_t code, int lane) {
  if (lane == 0 && out_T) {
    out_T[inst] = code;
  } else if (lane == 0) {
    fsched_metrics m;
    m.T = code;
    m.O = m.Q = m.E = m.C = m.W = 0;
    m.sum_completion = m.sum_latency = m.sum_extent = m.busy_steps = 0;
    m.peak_kv = m.unfair_steps = 0;
    m.max_extent = m.max_active = 0;
    out[inst] = m;
  }
}

template <int NW>
struct PoolBits {
  uint32_t w[NW];

  __device__ __forceinline__ void clear_all() {
#pragma unroll
    for (int i = 0; i < NW; ++i) w[i] = 0u;
  }
  // first set rank, -1 if none
  __device__ __forceinline__ int first() const {
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      uint64_t m = ballot(w[i] != 0u);
      if (m) {
        int L = __builtin_ctzll(m);
        uint32_t x = (uint32_t)readlane((int)w[i], L);
        return ((i * WAVE + L) << 5) + __builtin_ctz(x);
      }
    }
    return -1;
  }
  __device__ __forceinline__ void reset(int r, int lane) {
    int L = (r >> 5) & (WAVE - 1), wi = r >> 11;
    uint32_t b = 1u << (r & 31);
#pragma unroll
    for (int i = 0; i < NW; ++i)
      if (i == wi && lane == L) w[i] &= ~b;
  }
  // clear every rank <= r
  __device__ __forceinline__ void clear_upto(int r, int lane) {
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      int base = (i * WAVE + lane) << 5;
      if (base + 31 <= r) w[i] = 0u;
      else if (base <= r) w[i] &= ~((2u << (r - base)) - 1u);
    }
  }
  __device__ __forceinline__ int count() const {
    int c = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) c += __builtin_popcount(w[i]);
    return wave_sum(c);
  }
};

// Wave-uniform scalars of one instance.  At most 1,024 jobs of fewer than 2^20
// tokens run at once and their starts lie within 2^20 steps of each other, so
// the reservations, and every sum over the active jobs of (start - earliest
// start), of footprints or of footprint differences, stay below 2^31: they are
// held in 32 bits.  sum_s itself (and sp - sum_s) is kept modulo 2^32, and only
// differences of that kind are read from it.
struct SimState {
  int t, ndone, nact, min_s, max_s, min_end;
  int res;              // KV reservations of the active jobs (only with a KV budget: a
                        // plan run without one leaves them out, and no one reads them)
  uint32_t sum_s;       // summed start of the active jobs, modulo 2^32
  uint64_t sum_start;   // summed start of every admitted job
  // prefill variant: largest prompt - start and summed prompt of the active jobs
  // (the largest footprint at step t is t + G + 1)
  int G;
  uint32_t sp;
};

// acc += a * b, one 32 x 32 -> 64-bit multiply-add.
__device__ __forceinline__ void mac(uint64_t& acc, uint32_t a, uint32_t b) {
  acc += (uint64_t)a * b;
}

// Section 5 sums of the event-free spans.  Over a span of D steps with s active
// jobs, first largest footprint m0, externality xe per step and extent ext:
//   E += D xe; the largest footprints m0, m0 + 1, .. sum to D m0 + D (D - 1) / 2,
// kept doubled (SM2, and SSM2 times s) so that each is one product of 32-bit
// factors: s D < 2^30 and 2 m0 + D < 2^23.  The tokens held are largest at the
// span's last step: s (m0 + D - 1) - xe.
// The event loop is bound by instruction issue on both the vector and the
// scalar unit, and these sums are its largest scalar part: with 64-bit factors
// they took about 120 scalar instructions per event, now about 40 (65,536 x 2,000
// ISJL at B = 512: 6.23 -> 5.72 ms; 16,384 x 2,000 FCFS, where every completion
// is an event: 13.3 -> 10.9 ms).
struct SpanSums {
  uint64_t E, SM2, SSM2, X;
  uint32_t unfair, peak;
  __device__ __forceinline__ void clear() {
    E = SM2 = SSM2 = X = 0;
    unfair = peak = 0;
  }
  __device__ __forceinline__ void add(uint32_t D, uint32_t s, uint32_t m0, uint32_t xe, int ext,
                                      int alpha) {
    const uint32_t m2 = 2u * m0 + D - 1u;
    mac(E, D, xe);
    mac(SM2, D, m2);
    mac(SSM2, s * D, m2);
    mac(X, D, (uint32_t)ext);
    unfair += ext > alpha ? D : 0u;
    peak = max(peak, s * (m0 + D - 1u) - xe);
  }
};

// ROB: Robust-ISJL (Section 3.4): ordering, packs, caps and the KV reservation
// use prompt + the predicted upper bound of the output; each job still runs its
// true length, and fairness is checked on true progress.
// PRE: the prompt is prefilled at admission (Section 1 with eq. (1)'s decode
// progress): a job runs one step per output token, reserves prompt + output and
// its footprint in the batch cost is prompt + progress; fairness stays on
// progress.  The drain, A_max and fill sweeps are off; a release sweep of its own
// (up to 8 slots per lane) folds up to 64 completions in, ISJL with up to 2 slots
// per lane takes plan runs, and every other completion is an event.
// FILL: with the fill sweep (below).
// QH: ISJL with up to 8 slots per lane whose plan-queue links are in HBM
// scratch (else in LDS).  Every kernel with up to 8 slots per lane but FCFS's
// is held to 128 VGPRs, so that 4 waves share a SIMD where the LDS allows 16
// per CU.  FCFS's 4- and 8-slot kernels keep 3: with an event per completion
// they ran 13.4 ms at 3 and 14.6 at 4 (16,384 x 2,000 at B = 512).  With the fill
// sweep little is left between the two: 1.320 ms at 3, 1.304 at 4 (B = 256 1.198
// and 1.188; 4,096 x 2,000 at B = 200 538 and 535 us).
template <int POL, int K, int NW, bool ROB, bool PRE, bool FILL, bool QH = false,
          bool FAIR = false>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(K <= 2 || (K <= 8 && POL != POL_FCFS) ? 4 : (K <= 8 ? 3 : 1)))) void simulate_kernel(SimArgs a) {
  static_assert(!ROB || POL == POL_ISJL, "predicted sizes: ISJL only");
  static_assert(!FILL || (!ROB && !PRE && POL != POL_LJF), "fill sweep variants");
  extern __shared__ uint32_t lds_raw[];
  // With 4 or 8 slots per lane (but FCFS: 1.320 -> 1.345 ms at B = 512, 538 -> 558
  // us at B = 200) the wave's index in its block is taken into a scalar register:
  // every row pointer derived from the instance is then scalar, which is what
  // brings those kernels under 128 VGPRs.  With one slot per lane it shortens the
  // event loop's address chains (256 x 2,000 ISJL at B = 16: 918 -> 901 us).  With
  // two, ISJL's plan runs at a large finite alpha are slower with it, their scalar
  // registers being the scarcer ones (4,096 x 2,000 at B = 128: alpha = 256 399 ->
  // 404 us, 1024 1.11 -> 1.16 ms), the others 3 to 6 % faster (alpha = 16 216 ->
  // 209, infinite 368 -> 359, prompt prefilled 2,888 -> 2,728, LJF 149 -> 139).
  constexpr bool WIB_S = K <= 8 && K != 2 && POL != POL_FCFS;
  const int wib = WIB_S ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)
                        : (int)(threadIdx.x >> 6);
  const int64_t inst = (int64_t)blockIdx.x * (blockDim.x >> 6) + wib;
  if (inst >= a.n_inst) return;
  const int lane = lane_id();
  const int n = a.n;
  uint32_t* W = lds_raw + (size_t)wib * (size_t)a.wave_words;
  uint16_t* QN = (uint16_t*)(W + a.off_q);
  // ISJL with up to 8 slots per lane: the plan-queue links live in HBM scratch
  // when that lets more waves share a CU (agent-scope accesses, so one lane's
  // link is seen by the others), else in LDS; the launch picks the kernel for
  // the place (a branch on it at every link would cost the event loop more)
  constexpr bool QGLOBAL = POL == POL_ISJL && K <= 8 && QH;
  uint32_t* QG = QGLOBAL ? a.qlink + inst * (int64_t)a.q_stride : nullptr;
  auto qn_set = [&](int r, uint32_t v) {
    if constexpr (QGLOBAL) __hip_atomic_store(QG + r, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else QN[r] = (uint16_t)v;
  };
  auto qn_get = [&](int r) -> uint32_t {
    if constexpr (QGLOBAL) return __hip_atomic_load(QG + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else return QN[r];
  };
  uint16_t* STG = (uint16_t*)(W + a.off_stage);
  // Released ranks on their way into the bitmap (not FCFS); shares the gather
  // buffer, which is dead while releases are processed.
  uint32_t* PEND = W + a.off_stage;
  const int64_t row = inst * (int64_t)n;
  const int32_t* A = a.arrival + row;
  const int32_t* P = a.prompt + row;
  const int32_t* O = a.output + row;
  const int32_t* U = ROB ? a.upper + row : nullptr;  // predicted upper bounds of the outputs
  // true service length of job j (ROB: the length that plans used was larger)
  auto true_len = [&](int j, int plan) -> int {
    return ROB ? (PRE ? O[j] : P[j] + O[j]) : plan;
  };
  // KV reservation of job j planned with size `plan`
  auto resv_len = [&](int j, int plan) -> int { return PRE ? P[j] + plan : plan; };

  // ---- load, validate, instance constants --------------------------------
  // One pass over the job table: validation, instance totals and the
  // priority keys (LJF / ISJL: (-len, index); SJF: (len, index); FCFS:
  // (len, index) in job order, which is its release order when the arrivals
  // are sorted); padding keys sort last.
  const int NP = a.NP;
  int bad = 0, big = 0, late = 0, maxlen = 0, maxfoot = 0, maxarr = 0;
  int64_t osum = 0, qsum = 0, rsum = 0;
  int64_t lsum = 0;  // PRE: summed service length (else osum)
  uint64_t q2 = 0;  // twice the footprint sum Q: one 32 x 32 -> 64 product per job
  int carry_ar = 0;
  // The rows are software-pipelined: the loads of row r + PF are issued
  // while row r is processed, so PF rows of loads are in flight (clamped
  // indices keep every load in bounds; the rows past NP are never used).
  constexpr int PF = 4;
  int pf_a[PF], pf_p[PF], pf_o[PF], pf_u[PF];
#pragma unroll
  for (int d = 0; d < PF; ++d) {
    const int ic = min(d * WAVE + lane, n - 1);
    pf_a[d] = A[ic];
    pf_p[d] = P[ic];
    pf_o[d] = O[ic];
    pf_u[d] = ROB ? U[ic] : 0;
  }
  for (int r0 = 0; r0 < NP; r0 += PF * WAVE) {
#pragma unroll
  for (int d = 0; d < PF; ++d) {
    const int i0 = r0 + d * WAVE;
    if (i0 >= NP) break;
    const int i = i0 + lane;
    const bool in = i < n;
    const int ar0 = pf_a[d], p0 = pf_p[d], o0 = pf_o[d], u0 = ROB ? pf_u[d] : o0;
    {
      const int ic = min(i + PF * WAVE, n - 1);
      pf_a[d] = A[ic];
      pf_p[d] = P[ic];
      pf_o[d] = O[ic];
      if (ROB) pf_u[d] = U[ic];
    }
    const int ar = in ? ar0 : 0x7FFFFFFF, p = in ? p0 : 0, o = in ? o0 : 1;
    const int u = in ? u0 : o;
    int prev = __shfl_up(ar, 1);
    if (lane == 0) prev = i0 > 0 ? carry_ar : ar;
    carry_ar = readlane(ar, WAVE - 1);
    uint32_t key = 0xFFFFFFFFu;
    if (in) {
      bad |= (ar < 0) | (p < 0) | (o < 1) | (u < o);
      // service length, planning size and largest footprint
      const int64_t len = PRE ? (int64_t)o : (int64_t)p + (int64_t)o;
      const int64_t plan_len = PRE ? (int64_t)u : (int64_t)p + (int64_t)u;
      const int64_t foot = (int64_t)p + (int64_t)u;
      big |= (foot >= LEN_LIMIT);
      late |= (prev > ar);
      if (foot < LEN_LIMIT && len > maxlen) maxlen = (int)len;
      if (foot < LEN_LIMIT && foot > maxfoot) maxfoot = (int)foot;
      if (ar > maxarr) maxarr = ar;
      osum += (int64_t)p + (int64_t)o;  // tokens served
      // Q: the footprint summed over the job's own steps (Section 5), doubled:
      // len (len + 1), or o (2 p + o + 1) with the prompt prefilled; both
      // factors are below 2^22 in every instance that is simulated (a larger
      // footprint returns the too-large marker before Q is used)
      q2 += PRE ? (uint64_t)(uint32_t)o * (uint32_t)(2 * p + o + 1)
                : (uint64_t)(uint32_t)len * (uint32_t)(len + 1);
      rsum += ar;
      if (PRE) lsum += o;
      const uint32_t l32 = (uint32_t)(ROB ? plan_len : len) & LMASK;
      if (POL == POL_LJF || POL == POL_ISJL) key = ((LMASK - l32) << 12) | (uint32_t)i;
      else key = (l32 << 12) | (uint32_t)i;
    }
    W[i] = key;
  }
  }
  bad = ballot(bad != 0) != 0;
  big = ballot(big != 0) != 0;
  const bool unsorted = ballot(late != 0) != 0;  // the arrivals are not sorted by job index
  if (bad) {
    write_marker(a.out, a.out_T, inst, FSCHED_T_INVALID, lane);
    return;
  }
  if (big) {
    write_marker(a.out, a.out_T, inst, FSCHED_T_TOOLARGE, lane);
    return;
  }
  maxlen = wave_max(maxlen);
  maxfoot = wave_max(maxfoot);
  maxarr = wave_max(maxarr);
  osum = wave_sum64(osum);
  qsum = (int64_t)((uint64_t)wave_sum64((int64_t)q2) >> 1);  // every term is even
  rsum = wave_sum64(rsum);
  lsum = PRE ? wave_sum64(lsum) : osum;
  if (unsorted && maxarr >= ARR_LIMIT) {
    write_marker(a.out, a.out_T, inst, FSCHED_T_TOOLARGE, lane);
    return;
  }
  {
    // Largest makespan any policy here can reach: all work serialised after the
    // last release, plus one delayed plan start (<= alpha) per job.
    double amin = a.alpha < maxlen ? (double)a.alpha : (double)maxlen;
    double tb = (double)maxarr + (double)osum + (double)n * amin + 1.0;
    if (tb >= 2147483000.0) {
      write_marker(a.out, a.out_T, inst, FSCHED_T_TOOLARGE, lane);
      return;
    }
    double cb = (double)a.c * tb + (double)a.tau * (double)osum * (double)maxfoot;
    double wb = (double)a.c * tb + (double)a.tau * tb * (double)maxfoot;
    if (cb > 4.0e18 || wb > 4.0e18) {
      write_marker(a.out, a.out_T, inst, FSCHED_T_RANGE, lane);
      return;
    }
  }

  // ---- priority order -----------------------------------------------------
  uint16_t* RK = POL != POL_FCFS ? a.rank + inst * (int64_t)a.rank_stride : nullptr;
  if (POL == POL_FCFS && unsorted) {  // FCFS's order is the release order
    for (int i = lane; i < NP; i += WAVE)
      W[i] = i < n ? ((uint32_t)A[i] << 12) | (uint32_t)i : 0xFFFFFFFFu;
  }
  if (POL != POL_FCFS || unsorted) {
    wave_lds_sync();
    if constexpr (NW == 2) {  // more than 2,048 jobs
      wave_reg_sort<64, true>(W, lane);
    } else {
      switch (NP) {
        case 64: wave_reg_sort<1, true>(W, lane); break;
        case 128: wave_reg_sort<2, true>(W, lane); break;
        case 256: wave_reg_sort<4, true>(W, lane); break;
        case 512: wave_reg_sort<8, true>(W, lane); break;
        case 1024: wave_reg_sort<16, true>(W, lane); break;
        default: wave_reg_sort<32, true>(W, lane); break;
      }
    }
    wave_lds_sync();
    // each job's rank goes to the rank table for the release chunks (only this
    // wave touches its row); the keys come from their bank-free places, two blocks
    // of 32 at a time, which are rewritten in order once read
    for (int r = lane; r < n; r += WAVE) {
      uint32_t key = W[swz(r)];
      int id = (int)(key & 0xFFFu);
      uint32_t len;
      if (POL == POL_LJF || POL == POL_ISJL) len = LMASK - (key >> 12);
      else if (POL == POL_SJF) len = key >> 12;
      else len = (uint32_t)(PRE ? O[id] : P[id] + O[id]);
      W[r] = (len << 12) | (uint32_t)id;
      if (POL != POL_FCFS) RK[id] = (uint16_t)r;
    }
  }
  if (POL != POL_FCFS) {
    __threadfence_block();  // the stores complete before the row is read
    if (unsorted) {
      // the table is put in release order: one more sort per instance, after
      // which releases are taken a chunk at a time as with sorted arrivals
      // (4,095 x 1,333 ISJL at B = 64 in random job order: 0.35 ms; a second
      // launch that searched the unreleased ranks at every release took 0.87)
      if constexpr (NW == 2) {  // more than 2,048 jobs
        release_order<64>(A, RK, n, lane);
      } else {
        switch (NP) {
          case 64: release_order<1>(A, RK, n, lane); break;
          case 128: release_order<2>(A, RK, n, lane); break;
          case 256: release_order<4>(A, RK, n, lane); break;
          case 512: release_order<8>(A, RK, n, lane); break;
          case 1024: release_order<16>(A, RK, n, lane); break;
          default: release_order<32>(A, RK, n, lane); break;
        }
      }
      __threadfence_block();
    }
  }
  wave_lds_sync();

  // ---- state ---------------------------------------------------------------
  const int Beff = a.Beff;
  const int alpha = a.alpha;
  // reservations stay below 2^30, so a larger budget never binds
  const int M = a.M < (int64_t)IDLE ? (int)a.M : IDLE;
  int ws_start[K], ws_end[K];
  int ws_plan[K];  // ROB: KV reservation of the running job (from its planning size)
  int ws_p[K];     // PRE: prompt of the running job (its footprint offset)
  uint32_t ws_q[K];
  uint32_t ws_qn[K];  // links in HBM: the link of the queue's head, loaded ahead
  bool valid[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    ws_plan[k] = 0;
    ws_p[k] = 0;
    ws_start[k] = IDLE;
    ws_end[k] = IDLE;
    ws_q[k] = QNONE | (QNONE << 16);
    ws_qn[k] = QNONE;
    valid[k] = (k * WAVE + lane) < Beff;
  }
  PoolBits<NW> pool;
  pool.clear_all();
  int relk = 0;           // release cursor
  int qcount = 0;         // queued jobs: released, not admitted, not planned
  int chunk = -1;         // release chunk loaded in rel_t / rel_r
  int rel_t = IDLE, rel_r = 0;
  int rel_nx = IDLE;      // release of the first job after the loaded chunk
  int head = 0;           // FCFS: first waiting rank
  // ISJL
  int mode = 0;           // 0 FILL, 1 DRAIN
  int planned = 0;        // planned jobs not yet started
  int t_w1 = 0;           // earliest start of worker 0's planned job

  SimState S;
  S.t = 0;
  S.ndone = 0;
  S.nact = 0;
  S.min_s = IDLE;
  S.max_s = -1;
  S.min_end = IDLE;
  S.res = 0;
  S.sum_s = 0;
  S.sum_start = 0;
  S.G = -IDLE;
  S.sp = 0;
  // C = c T + tau sum_t |S_t| m_t and W = c T + tau sum_t m_t (m_t: the largest
  // footprint at step t, 0 when idle): c and tau are applied once at the end
  // (every step 0 .. T-1 is accounted exactly once)
  SpanSums acc;
  acc.clear();
  int acc_busy = 0, acc_maxext = 0, acc_maxact = 0;  // every makespan is below 2^31
  // With up to 2 slots per lane the sweeps' per-lane partial sums (and the
  // largest footprint) of their span terms carry over from sweep to sweep and
  // are summed over the wave once after the event loop: integer sums, so the
  // deferral changes no result, and a sweep ends without a reduction.  The
  // wider kernels have no registers to spare for them and reduce per sweep.
  constexpr bool DEFER = K <= 2;
  constexpr bool PLAN_RUN = POL == POL_ISJL && !FILL && K <= 2;
  SpanSums lane_sums;
  lane_sums.clear();
  auto reduce_lane_sums = [&](const SpanSums& l) {
    acc.E += (uint64_t)wave_sum64((int64_t)l.E);
    acc.SM2 += (uint64_t)wave_sum64((int64_t)l.SM2);
    acc.SSM2 += (uint64_t)wave_sum64((int64_t)l.SSM2);
    acc.X += (uint64_t)wave_sum64((int64_t)l.X);
    acc.unfair += (uint32_t)wave_sum((int)l.unfair);
    acc.peak = max(acc.peak, (uint32_t)wave_max((int)l.peak));  // below 2^31
  };
  int32_t* st_out = a.start ? a.start + row : nullptr;
  int32_t* fi_out = a.finish ? a.finish + row : nullptr;
  const int iter_max = 8 * n + 64;
  int iter = 0;
  bool failed = false;

  // Load release chunk `c`: 64 consecutive jobs in release order.
  auto load_chunk = [&](int c) {
    const int j = c * WAVE + lane;
    rel_t = IDLE;
    rel_r = 0;
    if (POL == POL_FCFS) {
      if (j < n) rel_t = A[unsorted ? pid(W[j]) : j];
      rel_r = j;
    } else if (j < n) {
      rel_r = RK[j];
      rel_t = A[unsorted ? pid(W[rel_r]) : j];
    }
    // (not looked up for unsorted arrivals: the chunk's last release step is
    // taken to go on after it)
    const int jn = (c + 1) * WAVE;
    rel_nx = jn >= n ? IDLE : (unsorted ? readlane(rel_t, WAVE - 1) : uni(A[jn]));
    chunk = c;
  };

  // Schedule output of one admitted job.
  auto emit = [&](int id, int t, int len) {
    if (st_out) st_out[id] = t;
    if (fi_out) fi_out[id] = t + len;
  };

  // Whether the first queued job (in priority order) cannot join the running
  // ones under the KV budget: then a strict-prefix admission admits nothing,
  // and the gather is skipped.  Checked with up to 4 slots per lane (B <= 256),
  // where a blocked head is common and the gather is a large share of an event;
  // the 8- and 16-slot kernels (at their register limit) gather regardless.
  auto head_blocked = [&]() -> bool {
    if (K > 4 || M == 0 || S.nact == 0) return false;
    const int r = pool.first();
    if (r < 0) return false;
    const uint32_t wv = W[r];
    return S.res + resv_len(pid(wv), plen(wv)) > M;
  };

  // The first G ranks of a bitmap (or all of them), in priority order, into
  // STG[0..); returns how many.  Each lane
  // writes its own word's ranks in turn; with up to 4 slots per lane, one bitmap
  // word per lane and more than 8 ranks, lane L instead finds the rank at
  // position c + L directly: the lane holding it by a binary search over the
  // lanes' inclusive counts, then the right set bit of that lane's word.
  auto gather_bits = [&](const PoolBits<NW>& bits, int G) __attribute__((always_inline)) -> int {
    if constexpr (K <= 4 && NW == 1) {
      if (G > 8) {
        const uint32_t x = bits.w[0];
        const int cnt = __builtin_popcount(x);
        const int incl = wave_scan_incl(cnt);
        G = min(G, readlane(incl, WAVE - 1));
        for (int c0 = 0; c0 < G; c0 += WAVE) {
          const int P = c0 + lane;
          int lo = 0;  // number of lanes whose count ends at or before P
#pragma unroll
          for (int step = WAVE / 2; step >= 1; step >>= 1) {
            const int v = __shfl(incl, lo + step - 1);
            if (v <= P) lo += step;
          }
          const int owner = lo < WAVE ? lo : WAVE - 1;
          uint32_t w = (uint32_t)__shfl((int)x, owner);
          int k = P - (__shfl(incl, owner) - __builtin_popcount(w));
          // the k-th set bit of w (k < popcount(w) for every P < G)
          int bit = 0;
#pragma unroll
          for (int half = 16; half >= 1; half >>= 1) {
            const int c = __builtin_popcount(w & ((1u << half) - 1u));
            if (k >= c) {
              k -= c;
              bit += half;
              w >>= half;
            }
          }
          if (P < G) STG[P] = (uint16_t)((owner << 5) + bit);
        }
        wave_lds_sync();
        return G;
      }
    }
    int gbase = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int cnt = __builtin_popcount(bits.w[i]);
      const int incl = wave_scan_incl(cnt);
      int pos = gbase + incl - cnt;
      uint32_t x = bits.w[i];
      const int base = (i * WAVE + lane) << 5;
      while ((x != 0u) & (pos < G)) {
        const int b = __builtin_ctz(x);
        x &= x - 1u;
        STG[pos] = (uint16_t)(base + b);
        pos++;
      }
      gbase += readlane(incl, 63);
    }
    wave_lds_sync();
    return min(G, gbase);
  };
  auto gather_first = [&](int G) __attribute__((always_inline)) { gather_bits(pool, G); };

  // Admit at step t the longest prefix of STG[0..G) that fits the KV budget
  // (strict order; a job that would run alone always fits), onto the first
  // eligible idle workers in index order (ISJL Phase TWO also needs an empty
  // plan queue).  Returns the number admitted.
  // Up to 64 jobs are read once, one per lane, and reach their slots through
  // lane shuffles, with up to 2 slots per lane and wherever the prompts have to
  // be looked up in the job table (16,384 x 2,000 with the prompt prefilled
  // 4.68 -> 4.54 ms, 4,096 x 1,000 SJF at B = 64 0.283 -> 0.267 ms).  Longer
  // batches, and the wide kernels without prompts (no gain there: 3.14 -> 3.15
  // ms at B = 512), read them from LDS again by slot.
  auto admit_prefix = [&](int t, int G, bool need_empty_queue, int& adm,
                          int& adm_minlen) __attribute__((always_inline)) -> int {
    if (K == 1 || ((K == 2 || PRE) && G <= WAVE)) {
      const int r = lane < G ? (int)STG[lane] : 0;
      const uint32_t wv = lane < G ? W[r] : 0u;
      const int id = pid(wv), plan = plen(wv);
      const int pp = (PRE && lane < G) ? P[id] : 0;
      const int len = (ROB && lane < G) ? true_len(id, plan) : plan;
      const int rv = plan + pp;  // reservation
      const int pre = wave_scan_incl(rv);
      int na = G;
      if (M != 0) {
        const uint64_t fm =
            ballot((lane < G) & ((lane > 0) | (S.nact > 0)) & (S.res + pre > M));
        if (fm) na = __builtin_ctzll(fm);
      }
      na = uni(na);
      if (na == 0) return 0;
      const bool inc = lane < na;
      if (inc) emit(id, t, len);
      int base = 0;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (base < na) {
          const bool el = valid[k] & (ws_end[k] == IDLE) &
                          (!need_empty_queue | ((ws_q[k] & 0xFFFFu) == QNONE));
          const uint64_t bm = ballot(el);
          const int idx = base + mbcnt(bm);
          const int src = min(idx, WAVE - 1);
          const int l2 = __shfl(len, src);
          const int r2 = (ROB || PRE) ? __shfl(rv, src) : 0, p2 = PRE ? __shfl(pp, src) : 0;
          if (el & (idx < na)) {
            ws_start[k] = t;
            ws_end[k] = t + l2;
            if (ROB || PRE) ws_plan[k] = r2;
            if (PRE) ws_p[k] = p2;
          }
          base += __builtin_popcountll(bm);
        }
      }
      // in priority order the shortest admitted job is the last (longest first)
      // or the first (SJF), by planning size
      adm_minlen = min(adm_minlen, ROB ? wave_min(inc ? len : IDLE)
                                       : readlane(len, POL == POL_SJF ? 0 : na - 1));
      if (PRE) {
        S.sp += (uint32_t)wave_sum(inc ? pp : 0);
        S.G = max(S.G, wave_max(inc ? pp : -IDLE) - t);  // na >= 1 jobs were admitted
      }
      pool.clear_upto(readlane(r, na - 1), lane);  // the first na queued ranks
      qcount -= na;
      adm += na;
      S.res += readlane(pre, na - 1);
      S.nact += na;
      return na;
    }
    int na = G;
    int ptot = -1;  // summed reservation of the admitted jobs, when the KV scan found it
    if (M != 0) {
      int run = S.res;
      for (int c0 = 0; c0 < G; c0 += WAVE) {
        const int j = c0 + lane;
        int len = 0;
        if (j < G) {
          const uint32_t wv = W[STG[j]];
          len = resv_len(pid(wv), plen(wv));
        }
        const int pre = wave_scan_incl(len);
        const bool fail = (j < G) & ((j > 0) | (S.nact > 0)) & (run + pre > M);
        const uint64_t fm = ballot(fail);
        if (fm) {
          const int f = __builtin_ctzll(fm);
          na = c0 + f;
          if (f > 0) run += readlane(pre, f - 1);
          break;
        }
        run += readlane(pre, 63);
      }
      ptot = run - S.res;
    }
    // the count in a scalar register, so the walk over the slot registers
    // below branches on it rather than masking lanes (measured on the kernels
    // with more than 2 slots per lane; the narrower ones ran no faster)
    if constexpr (K > 2) na = uni(na);
    if (na == 0) return 0;
    int base = 0, lplan = 0, lmin = IDLE, lp = 0, lpmax = -IDLE;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (base < na) {
        const bool el = valid[k] & (ws_end[k] == IDLE) &
                        (!need_empty_queue | ((ws_q[k] & 0xFFFFu) == QNONE));
        const uint64_t bm = ballot(el);
        const int idx = base + mbcnt(bm);
        if (el & (idx < na)) {
          const uint32_t wv = W[STG[idx]];
          const int plan = plen(wv);
          const int len = true_len(pid(wv), plan);
          ws_start[k] = t;
          ws_end[k] = t + len;
          emit(pid(wv), t, len);
          if (ROB || PRE) {
            const int rv = resv_len(pid(wv), plan);
            ws_plan[k] = rv;
            lplan += rv;
            lmin = min(lmin, len);
          } else {
            lplan += len;
          }
          if (PRE) {
            const int pp = P[pid(wv)];
            ws_p[k] = pp;
            lp += pp;
            lpmax = max(lpmax, pp);
          }
        }
        base += __builtin_popcountll(bm);
      }
    }
    if (ptot < 0) ptot = wave_sum(lplan);
    if (ROB || PRE) {
      adm_minlen = min(adm_minlen, wave_min(lmin));
    } else {
      // the gathered jobs are in priority order, so the shortest admitted one
      // is the last (longest first) or the first (SJF)
      adm_minlen = min(adm_minlen, plen(W[STG[POL == POL_SJF ? 0 : na - 1]]));
    }
    if (PRE) {
      S.sp += (uint32_t)wave_sum(lp);
      S.G = max(S.G, wave_max(lpmax) - t);  // na >= 1 jobs were admitted
    }
    pool.clear_upto(STG[na - 1], lane);  // the first na queued ranks
    qcount -= na;
    adm += na;
    S.res += ptot;
    S.nact += na;
    return na;
  };

  // Admit the first queued job if the KV budget lets it in (the usual case of one
  // completion freeing one worker): no gather and no scan.
  auto admit_one = [&](int t, bool need_empty_queue, int& adm, int& adm_minlen)
                       __attribute__((always_inline)) -> int {
    const int r = pool.first();
    const uint32_t wv = uniu(W[r]);
    const int id = pid(wv), plan = plen(wv);
    const int pp = PRE ? uni(P[id]) : 0;
    const int rv = plan + pp;
    if (M != 0 && S.nact > 0 && S.res + rv > M) return 0;
    const int len = ROB ? uni(true_len(id, plan)) : plan;
    if (lane == 0) emit(id, t, len);
    int at = -1;  // the first eligible worker
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if (at < 0) {
        const bool el = valid[k] & (ws_end[k] == IDLE) &
                        (!need_empty_queue | ((ws_q[k] & 0xFFFFu) == QNONE));
        const uint64_t bm = ballot(el);
        if (bm) at = k * WAVE + __builtin_ctzll(bm);
      }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const bool here = at == k * WAVE + lane;
      ws_start[k] = here ? t : ws_start[k];
      ws_end[k] = here ? t + len : ws_end[k];
      if (ROB || PRE) ws_plan[k] = here ? rv : ws_plan[k];
      if (PRE) ws_p[k] = here ? pp : ws_p[k];
    }
    adm_minlen = min(adm_minlen, len);
    if (PRE) {
      S.sp += (uint32_t)pp;
      S.G = max(S.G, pp - t);
    }
    pool.reset(r, lane);
    qcount -= 1;
    adm += 1;
    S.res += rv;
    S.nact += 1;
    return 1;
  };

  // Gather and admit the strict prefix of the first G queued jobs.  With up to 4
  // slots per lane and a binding KV budget, the first 8 are gathered and scanned
  // alone and the rest only if all 8 fit: admitting those 8 and then the prefix
  // of the next G - 8 is the same strict prefix, and a budget that stops early
  // spares the gather of all G.
  auto admit_first = [&](int t, int G, bool need_empty_queue, int& adm,
                         int& adm_minlen) __attribute__((always_inline)) -> int {
    constexpr int G0 = 8;
    if (K <= 2 && G == 1) return admit_one(t, need_empty_queue, adm, adm_minlen);
    if (K <= 4 && M != 0 && S.nact > 0 && G > G0) {
      gather_first(G0);
      const int na = admit_prefix(t, G0, need_empty_queue, adm, adm_minlen);
      if (na < G0) return na;
      gather_first(G - G0);
      return G0 + admit_prefix(t, G - G0, need_empty_queue, adm, adm_minlen);
    }
    gather_first(G);
    return admit_prefix(t, G, need_empty_queue, adm, adm_minlen);
  };

  // Section 5 sums of the next D steps with the active set as it is (not empty).
  // The largest footprint grows by one per step, and the span's externality is a
  // constant: each active job pays the largest footprint minus its own.
  auto account = [&](int D) {
    const uint32_t s = (uint32_t)S.nact;
    const uint32_t m0 = PRE ? (uint32_t)(S.t + S.G + 1) : (uint32_t)(S.t - S.min_s + 1);
    const uint32_t xe =
        PRE ? s * (uint32_t)S.G - (S.sp - S.sum_s) : S.sum_s - s * (uint32_t)S.min_s;
    const int ext = S.max_s - S.min_s;
    acc.add((uint32_t)D, s, m0, xe, ext, alpha);
    acc_busy += D;
    acc_maxext = max(acc_maxext, ext);
    acc_maxact = max(acc_maxact, S.nact);
  };

  // FAIR: launched when every wave of the grid is resident at once, so that the
  // launch lasts as long as its slowest wave.  A SIMD's arbiter issues for its
  // oldest wave first, which leaves the youngest to finish alone, one
  // dependent instruction at a time; turning each wave's priority with its
  // event count shares the issue slots among the SIMD's waves instead.
  int fair_turn = FAIR ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
  while (true) {
    int t = S.t;
    if constexpr (FAIR) {
      switch (fair_turn++ & 3) {
        case 0: __builtin_amdgcn_s_setprio(0); break;
        case 1: __builtin_amdgcn_s_setprio(1); break;
        case 2: __builtin_amdgcn_s_setprio(2); break;
        default: __builtin_amdgcn_s_setprio(3); break;
      }
    }
    // (1) retire the jobs whose last token was processed at t-1
    if (S.min_end == t) {
      // the earliest / latest start is searched again only if a job holding
      // it retires
      int nret = 0, lsum = 0, lplan = 0, lp = 0, me = IDLE;
      bool hmin = false, hmax = false, hG = false;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        const bool r = ws_end[k] == t;
        nret += __builtin_popcountll(ballot(r));
        if (r) {
          lsum += ws_end[k] - ws_start[k];
          if (ROB || PRE) lplan += ws_plan[k];
          if (PRE) {
            lp += ws_p[k];
            hG |= ws_p[k] - ws_start[k] == S.G;
          }
          hmin |= ws_start[k] == S.min_s;
          hmax |= ws_start[k] == S.max_s;
          ws_end[k] = IDLE;
          ws_start[k] = IDLE;
        }
        me = min(me, ws_end[k]);
      }
      int lret = wave_sum(lsum);
      S.min_end = wave_min(me);
      if (ballot(hmin)) {
        int mn = IDLE;
#pragma unroll
        for (int k = 0; k < K; ++k) mn = min(mn, ws_start[k]);
        S.min_s = wave_min(mn);
      }
      if (ballot(hmax)) {
        int mx = -1;
#pragma unroll
        for (int k = 0; k < K; ++k)
          if (ws_start[k] != IDLE) mx = max(mx, ws_start[k]);
        S.max_s = wave_max(mx);
      }
      if (PRE) {
        S.sp -= (uint32_t)wave_sum(lp);
        if (ballot(hG)) {
          int g = -IDLE;
#pragma unroll
          for (int k = 0; k < K; ++k)
            if (ws_end[k] != IDLE) g = max(g, ws_p[k] - ws_start[k]);
          S.G = wave_max(g);
        }
      }
      S.ndone += nret;
      S.nact -= nret;
      S.res -= (ROB || PRE) ? wave_sum(lplan) : lret;
      S.sum_s -= (uint32_t)nret * (uint32_t)t - (uint32_t)lret;
    }
    if (S.ndone == n) break;

    // (2) releases.  The jobs released by t are the next lanes of the loaded
    // chunk up to the first later arrival; their pool bits are scattered with
    // LDS atomics and folded into the register bitmap once.
    {
      bool any = false;
      while (relk < n) {
        if ((relk >> 6) != chunk) load_chunk(relk >> 6);
        const int off = relk & (WAVE - 1);
        const uint64_t late = ballot((lane >= off) & (rel_t > t));
        const int hi = late ? __builtin_ctzll(late) : WAVE;
        if (POL != POL_FCFS && hi > off) {
          if (!any) {
#pragma unroll
            for (int i = 0; i < NW; ++i) PEND[i * WAVE + lane] = 0u;
            wave_lds_sync();
            any = true;
          }
          if ((lane >= off) & (lane < hi)) atomicOr(&PEND[rel_r >> 5], 1u << (rel_r & 31));
          qcount += hi - off;
        }
        relk += hi - off;
        if (hi < WAVE) break;
      }
      if (POL != POL_FCFS && any) {
        wave_lds_sync();
#pragma unroll
        for (int i = 0; i < NW; ++i) pool.w[i] |= PEND[i * WAVE + lane];
        wave_lds_sync();
      }
    }

    // (3) A_max(t): largest progress among the jobs still active
    const int amax = S.nact > 0 ? t - S.min_s : 0;
    const int nact0 = S.nact;
    int adm = 0, adm_minlen = IDLE;
    bool kv_block = false;
    int free_empty = 0;  // ISJL: idle workers with nothing planned, after this step's admissions

    // (4) admissions
    if (POL == POL_FCFS) {
      int cnt = min(relk - head, Beff - S.nact);
      int done = 0;
      while (done < cnt) {
        int c = min(WAVE, cnt - done);
        int r = head + done + lane;
        uint32_t wv = lane < c ? W[r] : 0u;
        int len = plen(wv), id = pid(wv);
        const int pp = (PRE && lane < c) ? P[id] : 0;  // prompt (prefill variant)
        int pre = wave_scan_incl(len + pp);            // reservations
        bool fit = (M == 0) | (S.res + pre <= M) |
                   ((S.nact == 0) & (done == 0) & (lane == 0));
        uint64_t fm = ballot((lane < c) & !fit);
        int take = fm ? __builtin_ctzll(fm) : c;
        if (take > 0) {
          int base = 0;
#pragma unroll
          for (int k = 0; k < K; ++k) {
            if (base < take) {
              bool idle = valid[k] & (ws_end[k] == IDLE);
              uint64_t bm = ballot(idle);
              int idx = base + mbcnt(bm);
              int src = min(idx, WAVE - 1);
              int l2 = __shfl(len, src), id2 = __shfl(id, src);
              const int p2 = PRE ? __shfl(pp, src) : 0;
              if (idle & (idx < take)) {
                ws_start[k] = t;
                ws_end[k] = t + l2;
                if (PRE) {
                  ws_p[k] = p2;
                  ws_plan[k] = p2 + l2;
                }
                emit(id2, t, l2);
              }
              base += __builtin_popcountll(bm);
            }
          }
          int tl = readlane(pre, take - 1);  // reservations admitted
          adm_minlen = min(adm_minlen, wave_min(lane < take ? len : IDLE));
          adm += take;
          if (PRE) {
            S.sp += (uint32_t)wave_sum(lane < take ? pp : 0);
            S.G = max(S.G, wave_max(lane < take ? pp : -IDLE) - t);
          }
          S.res += tl;
          S.nact += take;
        }
        done += take;
        if (take < c) break;
      }
      head += done;
    } else if (POL == POL_LJF || POL == POL_SJF) {
      if (POL == POL_SJF || S.nact == 0) {
        const int freew = Beff - S.nact;
        if (freew > 0) {
          const int kp = qcount;
          const int G = min(freew, kp);
          if (G > 0 && !head_blocked()) admit_first(t, G, false, adm, adm_minlen);
        }
      }
    } else {  // ISJL
      // Epoch: empty machine, nothing planned, jobs queued -> Phase ONE.
      if (S.nact == 0 && planned == 0) {
        int kp = qcount;
        if (kp > 0) {
          mode = 0;
          int G = min(Beff, kp);
          gather_first(G);  // longest first
          // lengths of the gathered jobs: job j in chunk j / 64, lane j % 64
          // (worker w's long job is gathered job w, in the same place)
          int glen[K];
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const int j = k * WAVE + lane;
            glen[k] = j < G ? plen(W[STG[j]]) : 0;
          }
          // Bp: largest prefix of the longest jobs that fits the KV budget
          int Bp = G;
          if (M != 0) {
            int run = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              if (k * WAVE < G && Bp == G) {
                const int j = k * WAVE + lane;
                // reservation of gathered job j (prefill variant: + prompt)
                const int rv = (PRE && j < G) ? glen[k] + P[pid(W[STG[j]])] : glen[k];
                const int pre = wave_scan_incl(rv);
                const uint64_t fm = ballot((j < G) & (j >= 1) & (run + pre > M));
                if (fm) Bp = k * WAVE + __builtin_ctzll(fm);
                else run += readlane(pre, 63);
              }
            }
            if (Bp < 1) Bp = 1;
          }
          const int o1 = readlane(glen[0], 0);
          const int o2 = kp > 1 ? readlane(glen[0], 1) : 0;
          if (kp > 1 && Bp > 1 && o2 > alpha) {
            // m = min{Bp, #{len > alpha}}: the lengths are non-increasing, so it
            // is the first gathered job with len <= alpha, capped at Bp
            int m = Bp;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              if (k * WAVE < Bp && m == Bp) {
                const int j = k * WAVE + lane;
                const uint64_t fm = ballot((j < Bp) & (glen[k] <= alpha));
                if (fm) m = min(Bp, k * WAVE + __builtin_ctzll(fm));
              }
            }
            if constexpr (K <= 4) m = uni(m);  // scalar (measured: the 8-slot kernel ran slower)
            const int beta = a.beta;
            int cap[K], room[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
              int w = k * WAVE + lane;
              // the long jobs' ranks, out of the gather buffer's way until
              // they are appended below
              ws_qn[k] = w < m ? (uint32_t)STG[w] : QNONE;
              if ((w >= 1) & (w < m)) {
                cap[k] = min(2 * alpha, o1 - glen[k] + beta);
              } else if ((w >= m) & (w < Bp)) {
                cap[k] = alpha;
              } else {
                cap[k] = -1;
              }
              room[k] = cap[k];
            }
            // the m long jobs are the first m queued ranks
            const int rlast = STG[m - 1];
            pool.clear_upto(rlast, lane);
            qcount -= m;
            planned += m;
            // Pack scan (Algorithm 3): remaining queued jobs in decreasing length;
            // each goes to the first spare worker with room, else to the long
            // worker of largest index with room; a job that fits nowhere stays.
            //
            // 64 candidates at a time are gathered, one per lane, and the workers
            // are filled one by one in that order, each with the candidates left,
            // longest first, that fit its room.  That is the same assignment:
            // whether a candidate goes to a worker depends only on the longer ones
            // that went there and on its having been refused by the workers before
            // it.  A step is then one ballot, a lane read and a subtraction (the
            // candidate-by-candidate scan chose among all workers at each step: 8
            // ballots at 8 slots per lane, and 590 cycles per step even at one);
            // the batch's links and bitmap bits are written together after it.
            // 16,384 x 2,000 with the prompt prefilled, 890 steps per instance:
            // 7.17 ms with a step per candidate straight from the bitmap, 5.73 from
            // gathered candidates, 4.66 worker by worker.
            const bool has_spare = uni(Bp) > m;
            auto largest_room = [&]() -> int {
              int rm = room[0];
#pragma unroll
              for (int k = 1; k < K; ++k) rm = max(rm, room[k]);
              return wave_max(rm);
            };
            PoolBits<NW> scan = pool;  // the ranks still to visit (queued, after rlast)
            int from = rlast + 1;
            while (from < n) {
              // the first rank from `from` on whose length fits the largest room
              // (lengths are non-increasing in rank)
              const int remmax = largest_room();
              if (remmax <= 0) break;
              const int span = n - from;
              const int sstep = (span + WAVE - 1) / WAVE;
              const int pr = from + lane * sstep;
              const uint64_t fm = ballot(pr < n && plen(W[pr]) <= remmax);
              int lo, hi;
              if (fm) {
                const int L1 = __builtin_ctzll(fm);
                hi = from + L1 * sstep;
                lo = L1 > 0 ? from + (L1 - 1) * sstep + 1 : from;
              } else {
                // after the last probe inside [from, n)
                lo = from + ((span - 1) / sstep) * sstep + 1;
                hi = n;
              }
              const int q = lo + lane;
              const uint64_t fm2 = ballot(q < hi && plen(W[q]) <= remmax);
              const int b = fm2 ? lo + __builtin_ctzll(fm2) : hi;
              if (b >= n) break;
              scan.clear_upto(b - 1, lane);
              const int cnt = gather_bits(scan, WAVE);
              if (cnt == 0) break;
              const int cr = lane < cnt ? (int)STG[lane] : 0;  // candidates: rank, length
              const int cl = lane < cnt ? plen(W[cr]) : 0;
              wave_lds_sync();  // the batch is out of the gather buffer
              int prev = (int)QNONE;  // the job before it in its worker's queue
              const uint64_t all = cnt < WAVE ? (1ull << cnt) - 1 : ~0ull;
              uint64_t left = all;
              // worker w = k * 64 + b takes what fits, in order
              auto fill_worker = [&](int& room_k, uint32_t& q_k, int b) {
                int rm = readlane(room_k, b);
                const uint32_t qq = (uint32_t)readlane((int)q_k, b);
                int head_r = (int)(qq & 0xFFFFu), tail_r = (int)(qq >> 16);
                uint64_t m_fit = ballot(cl <= rm) & left;
                do {
                  const int i = __builtin_ctzll(m_fit);
                  rm -= readlane(cl, i);
                  const int r = readlane(cr, i);
                  prev = lane == i ? tail_r : prev;
                  tail_r = r;
                  if (head_r == (int)QNONE) head_r = r;
                  left &= ~(1ull << i);
                  m_fit &= m_fit - 1;  // those after it that still fit
                  m_fit &= ballot(cl <= rm);
                } while (m_fit);
                room_k = lane == b ? rm : room_k;
                q_k = lane == b ? (uint32_t)head_r | ((uint32_t)tail_r << 16) : q_k;
              };
              // the workers that fit the shortest candidate left (so each takes one)
              auto shortest = [&]() -> int { return readlane(cl, 63 - __builtin_clzll(left)); };
              // Several workers at once, up to 2 slots per lane: while each next
              // worker (of ws, in lane order or from the last) has an empty queue,
              // fits the next candidate and then has no room left for the
              // shortest, the i-th of them takes the i-th candidate and nothing
              // else (nearly every step at B = 16 and 128: 256 x 2,000 905 ->
              // 853 us, 4,096 x 2,000 451 -> 421 us).
              auto fill_run = [&](int& room_k, uint32_t& q_k, uint64_t& ws, bool up, int sh)
                                  __attribute__((always_inline)) -> bool {
                const int i1 = __builtin_ctzll(left);
                const uint64_t gap = ~(left >> i1);
                const int run = gap ? __builtin_ctzll(gap) : WAVE;
                const int j = up ? mbcnt(ws) : __builtin_popcountll(ws) - 1 - mbcnt(ws);
                const int src = min(max(i1 + j, 0), WAVE - 1);
                const int x = __shfl(cl, src), r = __shfl(cr, src);
                const uint64_t ok = ws & ballot((j < run) & (x <= room_k) & (room_k - x < sh) &
                                                ((q_k & 0xFFFFu) == QNONE));
                const uint64_t bad = ws & ~ok;
                uint64_t take = ok;
                if (bad)
                  take &= up ? (bad & -bad) - 1 : ~(~0ull >> __builtin_clzll(bad));
                const int g = __builtin_popcountll(take);
                if (g < 2) return false;
                const bool mine = (take >> lane) & 1ull;
                room_k -= mine ? x : 0;
                q_k = mine ? (uint32_t)r | ((uint32_t)r << 16) : q_k;
                left &= ~((g < WAVE ? (1ull << g) - 1 : ~0ull) << i1);
                ws &= ~take;
                return true;
              };
              if (has_spare) {  // spare workers, ascending
#pragma unroll
                for (int k = 0; k < K; ++k) {
                  const int w = k * WAVE + lane;
                  uint64_t ws = ballot((w >= m) & (w < Bp));
                  bool several = K <= 2;
                  while (ws && left) {
                    const int sh = shortest();
                    ws &= ballot(room[k] >= sh);
                    if (!ws) break;
                    if (K <= 2 && several) {
                      several = fill_run(room[k], ws_q[k], ws, true, sh);
                      if (several) continue;
                    }
                    const int b = __builtin_ctzll(ws);
                    ws &= ws - 1;
                    fill_worker(room[k], ws_q[k], b);
                  }
                }
              }
#pragma unroll
              for (int k = K - 1; k >= 0; --k) {  // long workers, largest index first
                const int w = k * WAVE + lane;
                uint64_t wl = ballot((w >= 1) & (w < m));
                bool several = K <= 2;
                while (wl && left) {
                  const int sh = shortest();
                  wl &= ballot(room[k] >= sh);
                  if (!wl) break;
                  if (K <= 2 && several) {
                    several = fill_run(room[k], ws_q[k], wl, false, sh);
                    if (several) continue;
                  }
                  const int b = 63 - __builtin_clzll(wl);
                  wl &= ~(1ull << b);
                  fill_worker(room[k], ws_q[k], b);
                }
              }
              const uint64_t placed = all & ~left;
              // the batch's links (a queue ends at its tail: the last one has none)
              // and its bits of the queued ranks
              const bool put = (placed >> lane) & 1ull;
              if (put & (prev != (int)QNONE)) qn_set(prev, (uint32_t)cr);
              const int np = __builtin_popcountll(placed);
              if (np > 0) {
#pragma unroll
                for (int w = 0; w < NW; ++w) PEND[w * WAVE + lane] = 0u;
                wave_lds_sync();
                if (put) atomicOr(&PEND[cr >> 5], 1u << (cr & 31));
                wave_lds_sync();
#pragma unroll
                for (int w = 0; w < NW; ++w) pool.w[w] &= ~PEND[w * WAVE + lane];
                wave_lds_sync();
                qcount -= np;
                planned += np;
              }
              if (cnt < WAVE) break;
              from = readlane(cr, WAVE - 1) + 1;
              scan.clear_upto(from - 1, lane);
            }
            // worker j in 2..M: its pack, then o_j; worker 1: o_1
            int pmax = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              int w = k * WAVE + lane;
              if ((w >= 1) & (w < Bp)) pmax = max(pmax, cap[k] - room[k]);
              const uint32_t r = ws_qn[k];
              if ((w >= 1) & (w < m)) {
                uint32_t h = ws_q[k] & 0xFFFFu, tl = ws_q[k] >> 16;
                if (tl != QNONE) qn_set((int)tl, r);
                else h = r;
                ws_q[k] = h | (r << 16);
              }
              if (w == 0) ws_q[k] = r | (r << 16);
            }
            wave_lds_sync();
            // HBM links: every store is done before a plan start reads them
            if constexpr (QGLOBAL) {
              __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
              // each head's link, loaded now for when it starts
#pragma unroll
              for (int k = 0; k < K; ++k) {
                const uint32_t h = ws_q[k] & 0xFFFFu;
                ws_qn[k] = h != (ws_q[k] >> 16) ? qn_get((int)h) : QNONE;
              }
            }
            pmax = wave_max(pmax);
            int idle1 = pmax - alpha;
            if (idle1 < 0) idle1 = 0;
            if (idle1 > alpha) idle1 = alpha;
            t_w1 = t + idle1;
          }
        }
      }
      // Plan starts (workers in index order), each guarded by
      // A_max(t) <= alpha and the KV budget.
      if (planned > 0 && amax <= alpha) {
        bool cand[K];
        int clen[K];
        uint32_t cwv[K];
        int csum = 0, ccnt = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
          int w = k * WAVE + lane;
          uint32_t h = ws_q[k] & 0xFFFFu;
          cand[k] = valid[k] & (ws_end[k] == IDLE) & (h != QNONE) & !((w == 0) & (t < t_w1));
          clen[k] = 0;  // reservation
          cwv[k] = 0u;
          if (cand[k]) {
            const uint32_t wv = W[h];
            cwv[k] = wv;
            clen[k] = resv_len(pid(wv), plen(wv));
          }
          csum += clen[k];
          ccnt += cand[k] ? 1 : 0;
        }
        int tot = wave_sum(csum);
        int ncand = wave_sum(ccnt);
        if (ncand > 0) {
          bool all = (M == 0) || (S.res + tot <= M) || (S.nact == 0 && ncand == 1);
          if (!all) {
            // Sequential KV check in worker order; a blocked worker waits and
            // later workers are still tried.
            int nk = 0;
            int rres = S.res;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              uint64_t mk = ballot(cand[k]);
              uint64_t keep = 0;
              while (mk) {
                int L = __builtin_ctzll(mk);
                mk &= mk - 1;
                int len = readlane(clen[k], L);
                if (S.nact + nk == 0 || rres + len <= M) {
                  keep |= 1ull << L;
                  rres += len;
                  nk++;
                }
              }
              cand[k] = cand[k] && ((keep >> lane) & 1ull);
            }
            tot = rres - S.res;
            ncand = nk;
          }
          int mlen = IDLE, lp = 0, lpmax = -IDLE;
#pragma unroll
          for (int k = 0; k < K; ++k) {
            if (cand[k]) {
              const uint32_t h = ws_q[k] & 0xFFFFu, tl = ws_q[k] >> 16;
              const uint32_t wv = cwv[k];
              const int plan = plen(wv);
              const int len = true_len(pid(wv), plan);
              ws_start[k] = t;
              ws_end[k] = t + len;
              if (ROB || PRE) ws_plan[k] = clen[k];
              if (PRE) {
                const int pp = clen[k] - plan;  // reservation less planning size
                ws_p[k] = pp;
                lp += pp;
                lpmax = max(lpmax, pp);
              }
              mlen = min(mlen, len);
              emit(pid(wv), t, len);
              uint32_t nx;
              if constexpr (QGLOBAL) {  // loaded ahead; the new head's link is loaded now
                nx = ws_qn[k];
                ws_qn[k] = (nx != QNONE) & (nx != tl) ? qn_get((int)nx) : QNONE;
              } else {
                nx = h != tl ? qn_get((int)h) : QNONE;
              }
              ws_q[k] = (nx == QNONE) ? (QNONE | (QNONE << 16)) : (nx | (ws_q[k] & 0xFFFF0000u));
            }
          }
          adm_minlen = min(adm_minlen, wave_min(mlen));
          adm += ncand;
          S.res += tot;
          if (PRE) {
            // the KV check may have dropped every candidate
            const int gm = wave_max(lpmax);
            if (gm != -IDLE) S.G = max(S.G, gm - t);
            S.sp += (uint32_t)wave_sum(lp);
          }
          S.nact += ncand;
          planned -= ncand;
        }
      }
      // Phase TWO (FILL): idle workers with nothing planned take the longest
      // queued unplanned job while A_max(t) <= alpha; otherwise DRAIN (until
      // the machine is empty, or with the resume reading until A_max <= alpha).
      if (mode == 1 && a.resume && amax <= alpha) mode = 0;
      if (mode == 0) {
        // idle workers with an empty plan queue (all idle ones when nothing is planned)
        int nie = Beff - S.nact;
        if (planned > 0) {
          nie = 0;
#pragma unroll
          for (int k = 0; k < K; ++k)
            nie += __builtin_popcountll(
                ballot(valid[k] & (ws_end[k] == IDLE) & ((ws_q[k] & 0xFFFFu) == QNONE)));
        }
        free_empty = nie;
        if (nie > 0) {
          const int kp = qcount;
          if (kp > 0) {
            if (amax > alpha) {
              mode = 1;
            } else if (head_blocked()) {
              kv_block = true;
            } else {
              const int G = min(nie, kp);
              const int na = admit_first(t, G, true, adm, adm_minlen);
              free_empty = nie - na;
              if (na < G) kv_block = true;
            }
          }
        }
      }
    }
    if (adm > 0) {
      S.sum_s += (uint32_t)adm * (uint32_t)t;
      mac(S.sum_start, (uint32_t)adm, (uint32_t)t);
      S.min_end = min(S.min_end, t + adm_minlen);
      if (nact0 == 0) S.min_s = t;
      S.max_s = t;
    }

    // Worker 1's planned job waits for its start time.
    const bool w0_timer = POL == POL_ISJL && planned > 0 && t_w1 > t &&
                          readlane(ws_end[0], 0) == IDLE &&
                          ((uint32_t)readlane((int)ws_q[0], 0) & 0xFFFFu) != QNONE;

    // Plan run (ISJL with jobs planned).  While every worker is busy, each
    // completion only starts the next planned job of its own worker, if the
    // guard and the KV budget allow: no release, queue or mode is read (a worker
    // left without a plan, a blocked start or worker 1's start time ends the
    // run, before the event).  The same holds with workers idle when Phase TWO
    // has stopped (DRAIN), or when it is held back by the KV budget: its first
    // job only gets longer by releases, so it stays blocked while the
    // reservations leave no room for the one queued now, up to the step where
    // A_max passes alpha.  Up to three quarters of the events with a binding alpha
    // are of this kind (4,096 x 2,000 at B = 128, alpha = 256: 593 -> 446 us; one
    // instance of 200 jobs at B = 50: 148 -> 111 us).  Up to 2 slots per lane: the
    // wide kernels ran no faster (3.13 ms at B = 512) or slower (4.51 -> 4.86 ms
    // with the prompt prefilled, 0.93 -> 0.99 ms with predicted sizes).  Not tried
    // with fewer than 4 jobs planned, where the run's set-up is not earned back
    // (from 1 on: 399 -> 406 us at alpha = 256, lognormal 4,096 x 1,000 at alpha =
    // 256 315 -> 319, though alpha = 64 232 -> 227; from 8 on 402, from 16 on 429,
    // and the one instance 54 -> 69 us on device arrays).
    if constexpr (PLAN_RUN) {
      const int spare = Beff - S.nact - (w0_timer ? 1 : 0);  // idle, but worker 1 on its timer
      const bool p2 = mode == 0 && spare > 0;
      if (planned >= 4 && S.nact > 0 && !(mode == 1 && a.resume) &&
          (!p2 || (!PRE && kv_block && qcount > 0))) {
        uint64_t held = 0;  // idle workers with a blocked planned job
#pragma unroll
        for (int k = 0; k < K; ++k) {
          uint64_t h = ballot(valid[k] & (ws_end[k] == IDLE) & ((ws_q[k] & 0xFFFFu) != QNONE));
          if (k == 0 && w0_timer) h &= ~1ull;
          held |= h;
        }
        if (!held) {
          const int p2len = p2 ? uni(plen(W[pool.first()])) : 0;
          while (true) {
            const int te = S.min_end;
            if ((w0_timer && te >= t_w1) || (p2 && te - S.min_s > alpha + 1)) break;
            int mn = IDLE;
            bool none = false;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              none |= (ws_end[k] == te) & ((ws_q[k] & 0xFFFFu) == QNONE);
              mn = min(mn, ws_end[k] == te ? IDLE : ws_start[k]);
            }
            if (ballot(none)) break;
            mn = wave_min(mn);
            if (mn == IDLE || te - mn > alpha) break;
            int ds = 0, dr = 0, cnt = 0;
            uint32_t wv[K];
#pragma unroll
            for (int k = 0; k < K; ++k) {
              const bool c = ws_end[k] == te;
              wv[k] = c ? W[ws_q[k] & 0xFFFFu] : 0u;
              const int rv = c ? resv_len(pid(wv[k]), plen(wv[k])) : 0;
              dr += c ? rv - ((ROB || PRE) ? ws_plan[k] : te - ws_start[k]) : 0;
              ds += c ? te - ws_start[k] : 0;
              cnt += __builtin_popcountll(ballot(c));
            }
            const int dres = M != 0 ? wave_sum(dr) : 0;
            if (M != 0 && (S.res + dres > M || (p2 && S.res + dres + p2len <= M))) break;
            account(te - S.t);
            S.sum_s += (uint32_t)wave_sum(ds);
            int me = IDLE, dp = 0, gm = -IDLE;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              if (ws_end[k] == te) {
                const uint32_t tl = ws_q[k] >> 16, h = ws_q[k] & 0xFFFFu;
                const int id = pid(wv[k]), plan = plen(wv[k]);
                const int len = true_len(id, plan);
                if (ROB || PRE) {
                  const int rv = resv_len(id, plan);
                  if (PRE) {
                    dp += (rv - plan) - ws_p[k];
                    ws_p[k] = rv - plan;
                  }
                  ws_plan[k] = rv;
                }
                ws_start[k] = te;
                ws_end[k] = te + len;
                emit(id, te, len);
                uint32_t nx;
                if constexpr (QGLOBAL) {  // loaded ahead, as in the planned starts
                  nx = ws_qn[k];
                  ws_qn[k] = (nx != QNONE) & (nx != tl) ? qn_get((int)nx) : QNONE;
                } else {
                  nx = h != tl ? qn_get((int)h) : QNONE;
                }
                ws_q[k] = nx == QNONE ? (QNONE | (QNONE << 16)) : (nx | (tl << 16));
              }
              me = min(me, ws_end[k]);
              if (PRE) gm = max(gm, ws_end[k] != IDLE ? ws_p[k] - ws_start[k] : -IDLE);
            }
            if (PRE) {
              S.sp += (uint32_t)wave_sum(dp);
              S.G = wave_max(gm);
            }
            S.min_s = mn;
            S.max_s = te;
            S.min_end = wave_min(me);
            S.res += dres;
            mac(S.sum_start, (uint32_t)cnt, (uint32_t)te);
            S.ndone += cnt;
            planned -= cnt;
            S.t = te;
            if (++iter > iter_max) break;
          }
          if (iter > iter_max) {
            failed = true;
            break;
          }
          // behind a blocked head the releases meanwhile are looked at first;
          // otherwise they matter no more than before
          if (p2 && S.t > t) continue;
          t = S.t;
        }
      }
    }

    // Release sweep (not LJF, which admits at an empty machine only; not with the
    // prompt prefilled, where the next completion is too close: 16,384 x 2,000
    // ISJL took 7.44 ms with it, 7.18 without).  With nothing queued and workers idle, every job
    // is admitted at its release, so a run of releases carries no decision as
    // long as all of them fit: the jobs of the loaded chunk, in release order,
    // up to the first one that finds no idle worker, exceeds the KV budget, or
    // comes at or after a completion (of an active job or of one admitted on
    // the way), worker 1's start time or the step where A_max passes alpha.  A
    // release step goes in as a whole or not at all (within one the policy's
    // order decides who waits).  Planned jobs of idle workers stay blocked
    // meanwhile: the KV budget only shrinks.  The spans between the release
    // steps have s = N + i + 1 active jobs after job i, with prefix sums of the
    // start offsets, and are summed one per lane.
    //
    // Event by event each release step costs the scatter into the bitmap, the
    // gather in priority order, the KV scan and the span sums; while the batch
    // fills (8 releases per step into 512 workers) those were 67 of 80 events per
    // instance: 65,536 x 2,000 ISJL at B = 512 5.69 -> 3.72 ms, 4,096 x 1,000 SJF
    // at B = 64 0.331 -> 0.287 ms.
    if constexpr (POL != POL_LJF && !PRE) {
      const int F = POL == POL_ISJL ? free_empty : Beff - S.nact;
      if ((POL == POL_FCFS ? head == relk : qcount == 0) && relk < n && S.nact > 0 && F > 0 &&
          (POL != POL_ISJL || mode == 0)) {
        if ((relk >> 6) != chunk) load_chunk(relk >> 6);
        const int off = relk & (WAVE - 1);
        int lim = S.min_end;  // releases before it
        if (w0_timer) lim = min(lim, t_w1);
        if (POL == POL_ISJL && alpha < maxlen) lim = min(lim, S.min_s + alpha + 1);
        if (readlane(rel_t, off) < lim) {
          const bool in = (lane >= off) & (rel_t < lim);
          const uint32_t wv = in ? W[rel_r] : 0u;
          const int id = pid(wv);
          const int len = in ? true_len(id, plen(wv)) : 0;
          const int rv = in ? resv_len(id, plen(wv)) : 0;
          const int end = in ? rel_t + len : IDLE;
          const int emin = wave_scan_incl_min(end);
          const int pre = wave_scan_incl(rv);
          const bool ok = in & (lane - off < F) & (rel_t < emin) & ((M == 0) | (S.res + pre <= M));
          const uint64_t bad = ballot(!ok & (lane >= off));
          const int cut = bad ? readlane(rel_t, __builtin_ctzll(bad)) : rel_nx;
          const int cnt = __builtin_popcountll(ballot(ok & (rel_t < cut)));
          if (cnt > 0) {
            const int last = off + cnt - 1;
            const bool inc = (lane >= off) & (lane <= last);
            const int t_last = readlane(rel_t, last);
            const int e_min = min(S.min_end, readlane(emin, last));
            // the next event: a completion, worker 1's start, or with a worker
            // left idle the next release
            int tn = e_min;
            if (w0_timer) tn = min(tn, t_w1);
            if (cnt < F) tn = min(tn, last + 1 < WAVE ? readlane(rel_t, last + 1) : rel_nx);
            const uint32_t xe0 = S.sum_s - (uint32_t)S.nact * (uint32_t)S.min_s;
            account(readlane(rel_t, off) - t);
            const int up = dpp<DPP_WAVE_SHL1>(rel_t, rel_t);
            const int dt = rel_t - S.min_s;
            const int pdt = wave_scan_incl(inc ? dt : 0);
            SpanSums here;
            here.clear();
            SpanSums& sums = DEFER ? lane_sums : here;
            if (inc & ((lane == last) | (up > rel_t)))
              sums.add((uint32_t)((lane == last ? tn : up) - rel_t),
                       (uint32_t)(S.nact + (lane - off) + 1), (uint32_t)(dt + 1),
                       xe0 + (uint32_t)pdt, dt, alpha);
            if constexpr (!DEFER) reduce_lane_sums(here);
            acc_busy += tn - readlane(rel_t, off);
            acc_maxext = max(acc_maxext, t_last - S.min_s);
            acc_maxact = max(acc_maxact, S.nact + cnt);
            if (inc) emit(id, rel_t, len);
            int base = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              if (base < cnt) {
                const bool el = valid[k] & (ws_end[k] == IDLE) &
                                (POL != POL_ISJL || (ws_q[k] & 0xFFFFu) == QNONE);
                const uint64_t bm = ballot(el);
                const int idx = base + mbcnt(bm);
                const int src = off + min(idx, cnt - 1);
                const int s2 = __shfl(rel_t, src), e2 = __shfl(end, src);
                const int r2 = ROB ? __shfl(rv, src) : 0;
                if (el & (idx < cnt)) {
                  ws_start[k] = s2;
                  ws_end[k] = e2;
                  if (ROB) ws_plan[k] = r2;
                }
                base += __builtin_popcountll(bm);
              }
            }
            const uint32_t sdt = (uint32_t)readlane(pdt, last);
            S.sum_s += (uint32_t)cnt * (uint32_t)S.min_s + sdt;
            mac(S.sum_start, (uint32_t)cnt, (uint32_t)S.min_s);
            S.sum_start += sdt;
            S.res += readlane(pre, last);
            S.nact += cnt;
            S.max_s = t_last;
            S.min_end = e_min;
            relk += cnt;
            if (POL == POL_FCFS) head = relk;
            S.t = tn;
            if (++iter > iter_max) {
              failed = true;
              break;
            }
            continue;
          }
        }
      }
    }

    // Release sweep with the prompt prefilled (not LJF; nothing planned).  Jobs run
    // their outputs only, so completions come between the releases: with nothing
    // queued neither carries a decision, and the completions of the jobs active
    // now are taken along.  The run of releases ends as in the sweep above
    // (counting no worker and no token that the completions free), or where a job
    // admitted on the way completes, and is taken when it has two release steps or
    // more, at most 64 completions, and some job active now outlasts it.  Releases
    // and sorted completions, one per lane each, are merged (a bitonic merge of
    // two registers) into at most 128 events; the jobs active after each event are
    // the others, the completions after it and the releases up to it: prefix sums,
    // a suffix maximum and a prefix maximum.  16,384 x 2,000 ISJL, where such steps
    // were some 130 of 324 events per instance: 4.59 -> 4.10 ms.  Not with 16 slots
    // per lane, where its registers leave one wave per SIMD instead of two: 2,048 x
    // 1,500 ISJL at B = 1000, alpha = 0 took 0.79 ms with it, 0.45 without.
    if constexpr (PRE && POL != POL_LJF && K <= 8) {
      const int F = Beff - S.nact;
      if ((POL == POL_FCFS ? head == relk : qcount == 0) && relk < n && S.nact > 1 && F > 0 &&
          (POL != POL_ISJL || (mode == 0 && planned == 0))) {
        if ((relk >> 6) != chunk) load_chunk(relk >> 6);
        const int off = relk & (WAVE - 1);
        int lim = IDLE;  // releases before it
        if (POL == POL_ISJL && alpha < maxlen) lim = S.min_s + alpha + 1;
        const int t1 = readlane(rel_t, off);
        const bool in = (lane >= off) & (rel_t < lim);
        const uint64_t in_m = ballot(in);
        if (t1 < lim && readlane(rel_t, 63 - __builtin_clzll(in_m)) > t1) {
          const uint32_t wv = in ? W[rel_r] : 0u;
          const int id = pid(wv);
          const int pp = in ? P[id] : 0;
          const int len = in ? (ROB ? true_len(id, plen(wv)) : plen(wv)) : 0;
          const int rv = in ? pp + plen(wv) : 0;
          const int end = in ? rel_t + len : IDLE;
          const int emin = wave_scan_incl_min(end);
          const int pre = wave_scan_incl(rv);
          const bool ok = in & (lane - off < F) & (rel_t < emin) & ((M == 0) | (S.res + pre <= M));
          const uint64_t bad = ballot(!ok & (lane >= off));
          const int cut = bad ? readlane(rel_t, __builtin_ctzll(bad)) : rel_nx;
          const int cnt = __builtin_popcountll(ballot(ok & (rel_t < cut)));
          const int last = off + max(cnt, 1) - 1;
          const int t_last = readlane(rel_t, last);
          int N0 = 0, hold = -1;  // completions by t_last; end of the latest started job
#pragma unroll
          for (int k = 0; k < K; ++k) {
            N0 += __builtin_popcountll(ballot(ws_end[k] <= t_last));
            hold = max(hold, ws_start[k] == S.max_s ? ws_end[k] : -1);
          }
          if (cnt > 1 && t_last > t1 && N0 <= WAVE && N0 < S.nact && wave_max(hold) >= t1) {
            const int N = S.nact;
            // the completions: end, progress and footprint (prompt + progress) at
            // t, packed into the lanes; largest ones of the other active jobs
            int ce = IDLE, cg = 0, ch = 0, rg = -1, rh = -IDLE, rend = IDLE;
            auto pack = [&](int what, int& to) __attribute__((always_inline)) {
              int base = 0;
#pragma unroll
              for (int k = 0; k < K; ++k) {
                const bool c = ws_end[k] <= t_last;
                const uint64_t bm = ballot(c);
                const int v = what == 0 ? ws_end[k] - t
                                        : (what == 1 ? t - ws_start[k] : ws_p[k] + t - ws_start[k]);
                if (c) PEND[base + mbcnt(bm)] = (uint32_t)v;
                base += __builtin_popcountll(bm);
              }
              wave_lds_sync();
              if (lane < N0) to = (int)PEND[lane];
              wave_lds_sync();
            };
            if (N0 > 0) {
              pack(0, ce);
              pack(1, cg);
              pack(2, ch);
            }
#pragma unroll
            for (int k = 0; k < K; ++k) {
              const bool o = (ws_end[k] != IDLE) & (ws_end[k] > t_last);
              rg = max(rg, o ? t - ws_start[k] : -1);
              rh = max(rh, o ? ws_p[k] + t - ws_start[k] : -IDLE);
              rend = min(rend, o ? ws_end[k] : IDLE);
            }
            rg = wave_max(rg);
            rh = wave_max(rh);
            rend = wave_min(rend);
            // events: time - t << 7 | release << 6 | lane (completions first)
            uint32_t ck[1] = {lane < N0 ? ((uint32_t)ce << 7) | (uint32_t)lane : 0xFFFFFFFFu};
            reg_sort_keys<1, true>(ck, lane);
            const int jl = min(off + lane, WAVE - 1);
            const int jt = __shfl(rel_t, jl);
            const uint32_t rk =
                lane < cnt ? ((uint32_t)(jt - t) << 7) | 64u | (uint32_t)jl : 0xFFFFFFFFu;
            const uint32_t rev = (uint32_t)__shfl((int)ck[0], (WAVE - 1) - lane);
            uint32_t ev0[1] = {min(rk, rev)}, ev1[1] = {max(rk, rev)};
            reg_sort_halves<1, true, WAVE / 2>(ev0, lane);
            reg_sort_halves<1, true, WAVE / 2>(ev1, lane);
            const int e_min = min(rend, readlane(emin, last));
            int tn = e_min;
            if (cnt - N0 < F)  // a worker is idle afterwards
              tn = min(tn, last + 1 < WAVE ? readlane(rel_t, last + 1) : rel_nx);
            const uint32_t ev[2] = {ev0[0], ev1[0]};
            const int first1 = readlane((int)ev1[0], 0);
            int tm[2], tx[2], dh[2], s[2], hs[2], hsuf[2], gsuf[2], hpre[2], lat[2];
            bool on[2], rel[2];
            // H: summed footprints at t
            const uint32_t H = (uint32_t)N * (uint32_t)t - S.sum_s + S.sp;
            int c_s = N, c_h = (int)H, c_hp = -IDLE, c_lat = S.max_s - t;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
              on[r] = ev[r] != 0xFFFFFFFFu;
              rel[r] = on[r] & ((ev[r] & 64u) != 0u);
              const int src = (int)(ev[r] & 63u);
              tm[r] = on[r] ? (int)(ev[r] >> 7) : tn - t;
              const int rp = __shfl(pp, src), xh = __shfl(ch, src), xg = __shfl(cg, src);
              const int hv = rp - tm[r];  // footprint at t of a job released here
              dh[r] = rel[r] ? hv : (on[r] ? -xh : 0);
              s[r] = c_s + wave_scan_incl(rel[r] ? 1 : (on[r] ? -1 : 0));
              hs[r] = c_h + wave_scan_incl(dh[r]);
              hpre[r] = max(c_hp, wave_scan_incl_max(rel[r] ? hv : -IDLE));
              lat[r] = max(c_lat, wave_scan_incl_max(rel[r] ? tm[r] : -IDLE));
              c_s = readlane(s[r], WAVE - 1);
              c_h = readlane(hs[r], WAVE - 1);
              c_hp = readlane(hpre[r], WAVE - 1);
              c_lat = readlane(lat[r], WAVE - 1);
              // of the completions after this event: suffix maxima, this register's
              // first (the later register's are added below)
              const bool com = on[r] & !rel[r];
              hsuf[r] = wave_scan_incl_max(__shfl(com ? xh : -IDLE, (WAVE - 1) - lane));
              gsuf[r] = wave_scan_incl_max(__shfl(com ? xg : -1, (WAVE - 1) - lane));
            }
            const int h1 = readlane(hsuf[1], WAVE - 1), g1 = readlane(gsuf[1], WAVE - 1);
            SpanSums here;
            here.clear();
            SpanSums& sums = DEFER ? lane_sums : here;
            int lmx = 0, lma = 0;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
              const int src = lane < WAVE - 1 ? (WAVE - 2) - lane : 0;
              int hq = __shfl(hsuf[r], src), gq = __shfl(gsuf[r], src);
              if (lane == WAVE - 1) hq = -IDLE, gq = -1;
              if (r == 0) hq = max(hq, h1), gq = max(gq, g1);
              hq = max(max(hq, rh), hpre[r]);
              gq = max(gq, rg);
              const int up = dpp<DPP_WAVE_SHL1>(tm[r], tm[r]);
              tx[r] = lane < WAVE - 1 ? up
                                      : (r == 0 && first1 != -1 ? (int)((uint32_t)first1 >> 7)
                                                                : tn - t);
              const int D = tx[r] - tm[r];
              if (on[r] & (D > 0)) {
                const int ext = lat[r] + gq;
                sums.add((uint32_t)D, (uint32_t)s[r], (uint32_t)(hq + tm[r] + 1),
                         (uint32_t)s[r] * (uint32_t)hq - (uint32_t)hs[r], ext, alpha);
                lmx = max(lmx, ext);
                lma = max(lma, s[r]);
              }
            }
            const int first = readlane(tm[0], 0);  // the first event
            account(first);
            if constexpr (!DEFER) reduce_lane_sums(here);
            acc_busy += tn - t - first;
            acc_maxext = max(acc_maxext, wave_max(lmx));
            acc_maxact = max(acc_maxact, wave_max(lma));
            const bool inc = (lane >= off) & (lane <= last);
            if (inc) emit(id, rel_t, len);
            mac(S.sum_start, (uint32_t)cnt, (uint32_t)t);
            S.sum_start += (uint32_t)wave_sum(inc ? rel_t - t : 0);
            // retire the completions, seat the admitted jobs
            int base = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              if (ws_end[k] <= t_last) {
                ws_end[k] = IDLE;
                ws_start[k] = IDLE;
              }
              const bool el = valid[k] & (ws_end[k] == IDLE);
              const uint64_t bm = ballot(el);
              const int idx = base + mbcnt(bm);
              const int src = off + min(idx, cnt - 1);
              const int s2 = __shfl(rel_t, src), e2 = __shfl(end, src);
              const int r2 = __shfl(rv, src), p2 = __shfl(pp, src);
              if (el & (idx < cnt)) {
                ws_start[k] = s2;
                ws_end[k] = e2;
                ws_plan[k] = r2;
                ws_p[k] = p2;
              }
              base += __builtin_popcountll(bm);
            }
            S.ndone += N0;
            S.nact = N - N0 + cnt;
            relk += cnt;
            if (POL == POL_FCFS) head = relk;
            {
              int lres = 0, mn = IDLE, gm = -IDLE;
              uint32_t ss = 0, sp = 0;
#pragma unroll
              for (int k = 0; k < K; ++k) {
                const bool act = ws_end[k] != IDLE;
                lres += act ? ws_plan[k] : 0;
                ss += act ? (uint32_t)ws_start[k] : 0u;
                sp += act ? (uint32_t)ws_p[k] : 0u;
                mn = min(mn, ws_start[k]);
                gm = max(gm, act ? ws_p[k] - ws_start[k] : -IDLE);
              }
              S.res = wave_sum(lres);
              S.sum_s = (uint32_t)wave_sum((int)ss);
              S.sp = (uint32_t)wave_sum((int)sp);
              S.min_s = wave_min(mn);
              S.G = wave_max(gm);
            }
            S.max_s = t_last;
            S.min_end = e_min;
            S.t = tn;
            if (++iter > iter_max) {
              failed = true;
              break;
            }
            continue;
          }
        }
      }
    }

    // Fill sweep (FCFS, SJF, and ISJL where alpha never binds, with nothing
    // planned; jobs queued).  Each coming completion admits the next jobs of the
    // queue's strict prefix that fit the freed slots and the KV budget.  While no
    // job admitted meanwhile completes and nothing is released, the admissions
    // follow from counts: the (at most 64) earliest completions are sorted, and
    // after those at positions <= p the first
    //   A(p) = min(G, free + p + 1, #{j : PQ_j <= M - res + RR_p})
    // queued jobs are in (PQ_j: summed reservations of the queued jobs 0..j in
    // priority order; RR_p: of the completed positions 0..p; A is
    // non-decreasing), and queued job j starts at the completion of the first
    // position with A(p) > j.  The spans are accounted in parallel as in the
    // drain sweep, with the other active jobs and the admitted ones added to the
    // suffix sums, up to the first completion or admitted job's completion that
    // the counts do not decide; the event loop takes it from there.  The last
    // group of the sorted completions is always left to the event loop, so every
    // counted event has a job of the sorted set still active.
    //
    // One position and one queued job per lane, however many slots a lane has:
    // an admitted job's completion ends the run after some tens of completions
    // (about 55 at B = 512 on the heavy-tailed workload), so sorting every active
    // job would cost more than it covers.  16,384 x 2,000 FCFS at B = 512, where
    // every completion was an event: 10.2 -> 1.32 ms.
    if constexpr (FILL) {
      const int Qn = POL == POL_FCFS ? relk - head : qcount;
      if (S.nact >= 2 && Qn > 0 && (POL != POL_ISJL || (mode == 0 && planned == 0))) {
        // completions before X: before the next release, and before the first
        // queued job could finish after being admitted at the first of them
        int X = IDLE;
        if (relk < n) {
          if ((relk >> 6) != chunk) load_chunk(relk >> 6);
          X = readlane(rel_t, relk & (WAVE - 1));
        }
        const int r0 = POL == POL_FCFS ? head : pool.first();
        X = min(X, S.min_end + plen(W[r0]));
        auto ends_before = [&](int x) -> int {
          int c = 0;
#pragma unroll
          for (int k = 0; k < K; ++k) c += __builtin_popcountll(ballot(ws_end[k] < x));
          return c;
        };
        int N0 = ends_before(X);  // completions sorted
        if constexpr (K > 1) {
          if (N0 > WAVE) {
            // an earlier X with at most 64 of them, by halving until 48 or more
            // are left (a halving costs K ballots, a short run a whole sweep).
            // Stopping at 24 or 32 took 1.49 and 1.57 ms for 16,384 x 2,000 FCFS
            // at B = 512, 48 1.32, 60 within 20 halvings 1.28; at B = 128 and 200,
            // where runs end early, 60 was slower (422 -> 429, 538 -> 547 us).
            int hi = X;
            X = S.min_end;
            N0 = 0;
            for (int i = 0; i < 10 && N0 < 48; ++i) {
              const int mid = X + ((hi - X) >> 1), c = ends_before(mid);
              if (c <= WAVE) {
                X = mid;
                N0 = c;
              } else {
                hi = mid;
              }
            }
          }
        }
        if (N0 >= 4) {
          const int N = S.nact;
          // completion - t and progress of the jobs that end before X, packed
          // into the lanes through the gather buffer with 2 or more slots; the
          // progress range of the others
          int e0 = IDLE, g0 = 0, rmax = -1, rmin = IDLE;
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const bool other = (ws_end[k] >= X) & (ws_end[k] != IDLE);
            rmax = max(rmax, other ? t - ws_start[k] : -1);
            rmin = min(rmin, other ? t - ws_start[k] : IDLE);
          }
          rmax = wave_max(rmax);
          rmin = wave_min(rmin);
          if constexpr (K == 1) {
            if (ws_end[0] < X) {
              e0 = ws_end[0] - t;
              g0 = t - ws_start[0];
            }
          } else {
            int base = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              const bool act = ws_end[k] < X;
              const uint64_t bm = ballot(act);
              if (act) PEND[base + mbcnt(bm)] = (uint32_t)(ws_end[k] - t);
              base += __builtin_popcountll(bm);
            }
            wave_lds_sync();
            if (lane < N0) e0 = (int)PEND[lane];
            wave_lds_sync();
            base = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              const bool act = ws_end[k] < X;
              const uint64_t bm = ballot(act);
              if (act) PEND[base + mbcnt(bm)] = (uint32_t)(t - ws_start[k]);
              base += __builtin_popcountll(bm);
            }
            wave_lds_sync();
            if (lane < N0) g0 = (int)PEND[lane];
            wave_lds_sync();
          }
          // sorted by completion: the lane rides in the low bits of the key
          // (completion - t is below 2^20)
          uint32_t key[1] = {e0 != IDLE ? ((uint32_t)e0 << 6) | (uint32_t)lane : 0xFFFFFFFFu};
          reg_sort_keys<1, true>(key, lane);
          const bool vq = lane < N0;
          const int e = vq ? (int)(key[0] >> 6) : IDLE;
          const int gs = __shfl(g0, (int)(key[0] & 63u));
          const int g = vq ? gs : 0;
          const int e_nx = dpp<DPP_WAVE_SHL1>(e, e);  // of the next position (IDLE past N0)
          // progress of the jobs active after this position but the admitted
          // ones: those above and the others
          const int gsum = (int)((uint32_t)N * (uint32_t)t - S.sum_s) - wave_scan_incl(g);
          int gmax = wave_scan_incl_max(__shfl(vq ? g : -1, (WAVE - 1) - lane));
          int gmin = wave_scan_incl_min(__shfl(vq ? g : IDLE, (WAVE - 1) - lane));
          {
            const int src = lane < WAVE - 1 ? (WAVE - 2) - lane : 0;
            gmax = __shfl(gmax, src);
            gmin = __shfl(gmin, src);
            gmax = max(lane < WAVE - 1 ? gmax : -1, rmax);
            gmin = min(lane < WAVE - 1 ? gmin : IDLE, rmin);
          }
          // queued job per lane: length, and summed reservations in priority order
          const int Gq = min(Qn, WAVE);
          if (POL != POL_FCFS) gather_first(Gq);
          const uint32_t qw =
              lane < Gq ? W[POL == POL_FCFS ? head + lane : (int)STG[lane]] : 0u;
          const int qlen = plen(qw);
          const int qsum_l = wave_scan_incl(qlen);
          const int pq = lane < Gq ? qsum_l : IDLE;
          // A: queued jobs admitted once the positions <= this one have completed
          const int room = Beff - N + lane + 1;
          int A = min(Gq, room);
          if (M != 0) {
            // lengths are the reservations
            const int b = M - (S.res - wave_scan_incl(vq ? e + g : 0));
            int lo = 0;  // queued jobs whose summed reservations fit
#pragma unroll
            for (int step = WAVE; step >= 1; step >>= 1) {
              const int x = __shfl(pq, min(lo + step, WAVE) - 1);
              if ((lo + step <= WAVE) & (x <= b) & (x != IDLE)) lo += step;
            }
            A = min(A, lo);
          }
          // more jobs than the gathered ones might be admitted
          const bool more = (Gq < Qn) & (A == Gq) & (room > Gq);
          const int ap = vq ? A : IDLE;
          if (!vq) A = 0;
          // start of queued job `lane` relative to t (IDLE: not admitted at these
          // positions), the earliest completion among jobs 0..lane and their
          // summed starts
          int sg;
          {
            int lo = 0;  // positions with A <= lane
#pragma unroll
            for (int step = WAVE; step >= 1; step >>= 1) {
              const int x = __shfl(ap, min(lo + step, WAVE) - 1);
              if ((lo + step <= WAVE) & (x <= lane)) lo += step;
            }
            const int es = __shfl(e, min(lo, WAVE - 1));
            sg = lo < N0 ? es : IDLE;
          }
          const int pm = wave_scan_incl_min(sg == IDLE ? IDLE : sg + qlen);
          const int sa = wave_scan_incl(sg == IDLE ? 0 : sg);
          // Which completions the counts decide: the event at group end q is
          // taken if no admitted job has completed by then; the span after it
          // ends early at an admitted job's completion.
          const int pmx = __shfl(pm, max(A - 1, 0)), sax = __shfl(sa, max(A - 1, 0)),
                    sgx = __shfl(sg, max(A - 1, 0));
          const int pmA = A > 0 ? pmx : IDLE;
          const uint64_t ge = ballot(vq & (e_nx > e));
          const uint64_t open = ge & ballot((lane + 1 >= N0) | (pmA <= e) | more);
          const uint64_t cut = ge & ~open & ballot(pmA < e_nx);
          // taken: the group ends below the first open one, up to the first cut one
          uint64_t taken = ge & (open ? (open & -open) - 1 : ~0ull);
          if (cut) taken &= (cut & -cut) | ((cut & -cut) - 1);
          const int p_m = taken ? 63 - __builtin_clzll(taken) : -1;
          const int e_first = readlane(e, 0);
          const int tau_rel = p_m >= 0 ? readlane(min(e_nx, pmA), p_m) : e_first;
          const int A_m = p_m >= 0 ? readlane(A, p_m) : 0;
          // spans after each counted event, with the jobs still active and the
          // admitted jobs 0..A-1
          SpanSums here;
          here.clear();
          SpanSums& sums = DEFER ? lane_sums : here;
          int lmx = 0, lma = 0;
          if ((taken >> lane) & 1u) {
            // starts relative to t: -gmax the earliest, sgx (of the last
            // admitted job) or -gmin the latest
            const int s = N - 1 - lane + A;
            const int ext = (A > 0 ? sgx : -gmin) + gmax;
            sums.add((uint32_t)((lane == p_m ? tau_rel : e_nx) - e), (uint32_t)s,
                     (uint32_t)(e + gmax + 1),
                     (uint32_t)(s * gmax - gsum + (A > 0 ? sax : 0)), ext, alpha);
            lmx = ext;
            lma = s;
          }
          account(e_first);  // span [t, first event): the jobs active now
          if constexpr (!DEFER) reduce_lane_sums(here);
          acc_busy += tau_rel - e_first;
          acc_maxext = max(acc_maxext, wave_max(lmx));
          acc_maxact = max(acc_maxact, wave_max(lma));
          // starts of the admitted jobs
          const bool adm_l = lane < A_m;
          mac(S.sum_start, (uint32_t)A_m, (uint32_t)t);
          if (A_m > 0) S.sum_start += (uint32_t)readlane(sa, A_m - 1);
          if (adm_l) emit(pid(qw), t + sg, qlen);
          // retire every job done by tau, then seat the admitted ones that are
          // still running
          const int tau = t + tau_rel;
          S.ndone += ends_before(tau + 1) + __builtin_popcountll(ballot(adm_l & (sg + qlen <= tau_rel)));
#pragma unroll
          for (int k = 0; k < K; ++k) {
            if (ws_end[k] <= tau) {
              ws_end[k] = IDLE;
              ws_start[k] = IDLE;
            }
          }
          if (A_m > 0) {
            int base = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              if (base < A_m) {
                const bool idle = valid[k] & (ws_end[k] == IDLE);
                const uint64_t bm = ballot(idle);
                const int idx = base + mbcnt(bm);
                const int jc = min(idx, A_m - 1);
                const int st = t + __shfl(sg, jc), en = st + __shfl(qlen, jc);
                if (idle & (idx < A_m) & (en > tau)) {
                  ws_start[k] = st;
                  ws_end[k] = en;
                }
                base += __builtin_popcountll(bm);
              }
            }
            if (POL == POL_FCFS) {
              head += A_m;
            } else {
              pool.clear_upto(STG[A_m - 1], lane);
              qcount -= A_m;
            }
          }
          {
            int cnt = 0, lres = 0, mn = IDLE, mx = -1, me = IDLE;
            uint32_t ss = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              const bool act = ws_end[k] != IDLE;
              cnt += __builtin_popcountll(ballot(act));
              lres += act ? ws_end[k] - ws_start[k] : 0;
              ss += act ? (uint32_t)ws_start[k] : 0u;
              mn = min(mn, ws_start[k]);
              mx = max(mx, act ? ws_start[k] : -1);
              me = min(me, ws_end[k]);
            }
            S.nact = cnt;
            S.res = wave_sum(lres);
            S.sum_s = (uint32_t)wave_sum((int)ss);
            S.min_s = wave_min(mn);
            S.max_s = wave_max(mx);
            S.min_end = wave_min(me);
          }
          S.t = tau;
          if (++iter > iter_max) {
            failed = true;
            break;
          }
          continue;
        }
      }
    }

    // Drain sweep.  LJF between batches and ISJL in DRAIN admit nothing through
    // Phase TWO, and a planned ISJL job can start only at a step where
    // A_max(t) <= alpha, which (A_max grows between completions) can first hold
    // right after a completion, or when the machine is empty.  Every completion
    // before that carries no decision: the active jobs are sorted by
    // completion (in registers) and each span between consecutive completions
    // is accounted in parallel, the jobs active after position i being the
    // positions > i (their count, progress sum and progress range are suffix
    // scans).  The sweep stops at the first completion after which a planned
    // job could start; the jobs still active there stay in their slots.
    // The same holds for FCFS, SJF and ISJL in FILL with nothing queued or
    // planned: no completion before the next release carries a decision, so
    // those completions are swept too (when there are a few of them).
    int quiet = 0;  // completions up to the next release, when nothing waits
    if (!PRE && POL != POL_LJF && S.nact > 0 &&
        (POL == POL_FCFS ? head == relk
                         : (qcount == 0 && (POL != POL_ISJL || (mode == 0 && planned == 0))))) {
      int r_next = IDLE;
      if (relk < n) {
        if ((relk >> 6) != chunk) load_chunk(relk >> 6);
        r_next = readlane(rel_t, relk & (WAVE - 1));
      }
      if (S.min_end <= r_next) {
#pragma unroll
        for (int k = 0; k < K; ++k)
          quiet += __builtin_popcountll(ballot((ws_end[k] != IDLE) & (ws_end[k] <= r_next)));
      }
    }
    // ISJL in FILL (or waiting on worker 1's timer) with A_max(t) > alpha: no
    // planned start, no Phase TWO admission and no epoch can come before the
    // first completion after which A_max <= alpha (A_max only grows between
    // completions, and every start needs it within alpha).  The only decision
    // meanwhile is Phase TWO's switch to DRAIN, at the first event with an idle
    // worker that has nothing planned and a queued job; both only appear over
    // the span, so it is settled from their first times after the sweep.  Taken
    // when at least two completions come before the last of the oldest active
    // jobs ends (A_max stays above alpha until then); compiled into the kernels
    // with up to 2 slots per lane (on the wider ones it did not fire on the
    // measured workloads and only added code).
    bool amax_sweep = false;
    if (POL == POL_ISJL && K <= 2 && !PRE && !FILL && S.nact > 0 && t - S.min_s > alpha &&
        !(mode == 1 && !w0_timer) && quiet < 3) {
      int oe = -1;
#pragma unroll
      for (int k = 0; k < K; ++k)
        if (ws_start[k] == S.min_s) oe = max(oe, ws_end[k]);
      oe = wave_max(oe);
      int before = 0;
#pragma unroll
      for (int k = 0; k < K; ++k) before += __builtin_popcountll(ballot(ws_end[k] < oe));
      amax_sweep = before >= 2;
    }
    bool sweep = !PRE &&
                 (POL == POL_LJF || (POL == POL_ISJL && mode == 1 && !w0_timer) || quiet >= 3 ||
                  amax_sweep) &&
                 S.nact > 0;
    if (sweep) {
      const int N = S.nact;
      // Progress is at most t - min_s and end - t at most the longest job:
      // when both fit one word together the progress rides in the low bits
      // of the key and the sort moves keys only.
      const int gbits = 32 - __builtin_clz((uint32_t)(t - S.min_s) | 1u);
      const bool packed = gbits < 32 && (int64_t)maxlen < (int64_t)(0xFFFFFFFFu >> gbits);
      int stop = 0, e0 = 0, st_g = 0, st_gmax = -1, st_gmin = IDLE, tau_end = 0;
      SpanSums here;
      here.clear();
      SpanSums& sums = DEFER ? lane_sums : here;
      // Sort the N completions into KS registers per lane (position
      // p = lane * KS + k holds the p-th) and account the spans.  KS = K sorts
      // every slot in place; KS = 1 first packs up to 64 active slots into one
      // register through the gather buffer (for K >= 4).
      auto sweep_body = [&](auto ks_tag) {
        constexpr int KS = decltype(ks_tag)::value;
        uint32_t dk[KS];  // end - t (unused positions: all ones, sorted last)
        int dg[KS];       // progress t - start, carried with its key
        if (packed) {
          if constexpr (KS == K) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
              const bool act = ws_end[k] != IDLE;
              dk[k] = act ? ((uint32_t)(ws_end[k] - t) << gbits) | (uint32_t)(t - ws_start[k])
                          : 0xFFFFFFFFu;
            }
          } else {
            int base = 0;
#pragma unroll
            for (int k = 0; k < K; ++k) {
              const bool act = ws_end[k] != IDLE;
              const uint64_t bm = ballot(act);
              if (act)
                PEND[base + mbcnt(bm)] =
                    ((uint32_t)(ws_end[k] - t) << gbits) | (uint32_t)(t - ws_start[k]);
              base += __builtin_popcountll(bm);
            }
            wave_lds_sync();
            dk[0] = lane < N ? PEND[lane] : 0xFFFFFFFFu;
            wave_lds_sync();
          }
          reg_sort_keys<KS, true>(dk, lane);
          const uint32_t gmask = (1u << gbits) - 1u;
#pragma unroll
          for (int k = 0; k < KS; ++k) {
            dg[k] = (int)(dk[k] & gmask);
            dk[k] = dk[k] == 0xFFFFFFFFu ? 0xFFFFFFFFu : dk[k] >> gbits;
          }
        } else if constexpr (KS == K) {
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const bool act = ws_end[k] != IDLE;
            dk[k] = act ? (uint32_t)(ws_end[k] - t) : 0xFFFFFFFFu;
            dg[k] = act ? t - ws_start[k] : 0;
          }
          reg_sort_payload<K>(dk, dg, lane);
        }
        // Suffix state of the lanes above this one (positions >= (lane+1)*KS):
        // progress sum, max and min.
        int xs_g, xs_max, xs_min;
        {
          int lg = 0, lmx = -1, lmn = IDLE;
#pragma unroll
          for (int k = 0; k < KS; ++k) {
            if (lane * KS + k < N) {
              lg += dg[k];
              lmx = max(lmx, dg[k]);
              lmn = min(lmn, dg[k]);
            }
          }
          const int incl = wave_scan_incl(lg);
          xs_g = readlane(incl, WAVE - 1) - incl;
          const int rmx = wave_scan_incl_max(__shfl(lmx, (WAVE - 1) - lane));
          const int rmn = wave_scan_incl_min(__shfl(lmn, (WAVE - 1) - lane));
          const int src = lane < WAVE - 1 ? (WAVE - 2) - lane : 0;
          xs_max = __shfl(rmx, src);
          xs_min = __shfl(rmn, src);
          if (lane == WAVE - 1) {
            xs_max = -1;
            xs_min = IDLE;
          }
        }
        // completion time of the first position of the next lane
        const int e_up = t + dpp<DPP_WAVE_SHL1>((int)dk[0], (int)dk[0]);
        // Stop position: the lowest position ending a tie group after which
        // the machine is empty or A_max <= alpha (A_max right after the
        // completions at e is e - t + the largest progress still active).
        stop = quiet >= 3 ? quiet - 1 : N - 1;
        if (POL == POL_ISJL && (planned > 0 || (a.resume && mode == 1) || amax_sweep)) {
          int cg_max = xs_max, lfound = IDLE;
#pragma unroll
          for (int k = KS - 1; k >= 0; --k) {
            const int pos = lane * KS + k;
            const bool valid = pos < N;
            const int e = t + (int)dk[k];
            const int e_next = (k + 1 < KS) ? t + (int)dk[k + 1 < KS ? k + 1 : k] : e_up;
            const bool group_end = valid & ((pos + 1 >= N) | (e_next > e));
            if (group_end & ((pos + 1 >= N) | (e - t + cg_max <= alpha))) lfound = pos;
            if (valid) cg_max = max(cg_max, dg[k]);
          }
          stop = min(stop, wave_min(lfound));
        }
        // Spans between consecutive completions below `stop`, each with the
        // jobs at the positions above (count N - 1 - p, progress suffix sums).
        int sg = 0, sgmax = -1, sgmin = IDLE, se = 0;
        {
          int cg = xs_g, cg_max = xs_max, cg_min = xs_min;
#pragma unroll
          for (int k = KS - 1; k >= 0; --k) {
            const int pos = lane * KS + k;
            const bool valid = pos < N;
            const int e = t + (int)dk[k];
            const int e_next = (k + 1 < KS) ? t + (int)dk[k + 1 < KS ? k + 1 : k] : e_up;
            if (valid & (pos < stop) & (e_next > e)) {
              const int s = N - 1 - pos;
              sums.add((uint32_t)(e_next - e), (uint32_t)s, (uint32_t)(e - t + cg_max + 1),
                       (uint32_t)(s * cg_max - cg), cg_max - cg_min, alpha);
            }
            if (pos == stop) {
              sg = cg;
              sgmax = cg_max;
              sgmin = cg_min;
              se = e;
            }
            if (valid) {
              cg += dg[k];
              cg_max = max(cg_max, dg[k]);
              cg_min = min(cg_min, dg[k]);
            }
          }
        }
        const int Ls = stop / KS;
        st_g = readlane(sg, Ls);
        st_gmax = readlane(sgmax, Ls);
        st_gmin = readlane(sgmin, Ls);
        tau_end = readlane(se, Ls);
        e0 = t + readlane((int)dk[0], 0);
      };
      if constexpr (K >= 4) {
        // the packing goes through the gather buffer: only when it holds 64 words
        if (packed && N <= WAVE && a.wave_words - a.off_stage >= WAVE)
          sweep_body(std::integral_constant<int, 1>{});
        else sweep_body(std::integral_constant<int, K>{});
      } else {
        sweep_body(std::integral_constant<int, K>{});
      }
      // span [t, e_0): every job still active; the set only shrinks after it,
      // so it also carries the largest extent and count of the sweep
      {
        account(e0 - t);
      }
      if constexpr (!DEFER) reduce_lane_sums(here);
      acc_busy += tau_end - e0;
      if (POL == POL_ISJL && amax_sweep && mode == 0) {
        // Phase TWO switches to DRAIN at the first event before tau_end with an
        // idle worker that has nothing planned (from its first completion, or
        // now) and a queued job (now, or from the next release)
        int tn_free = IDLE;
        if (planned == 0 && S.nact < Beff) {
          tn_free = t;
        } else {
          int fe = IDLE;
          bool idle_empty = false;
#pragma unroll
          for (int k = 0; k < K; ++k) {
            const bool empty_q = (ws_q[k] & 0xFFFFu) == QNONE;
            if (valid[k] & empty_q) {
              if (ws_end[k] == IDLE) idle_empty = true;
              else fe = min(fe, ws_end[k]);
            }
          }
          tn_free = ballot(idle_empty) ? t : wave_min(fe);
        }
        int tn_queued = IDLE;
        if (qcount > 0) {
          tn_queued = t;
        } else if (relk < n) {
          if ((relk >> 6) != chunk) load_chunk(relk >> 6);
          tn_queued = readlane(rel_t, relk & (WAVE - 1));
        }
        if (max(tn_free, tn_queued) < tau_end) mode = 1;
      }
      // retire every job that completed by tau_end
      int rc = 0, rl = 0, me = IDLE;
#pragma unroll
      for (int k = 0; k < K; ++k) {
        if (ws_end[k] <= tau_end) {
          rc++;
          rl += ROB ? ws_plan[k] : ws_end[k] - ws_start[k];
          ws_end[k] = IDLE;
          ws_start[k] = IDLE;
        }
        me = min(me, ws_end[k]);
      }
      const int nret = wave_sum(rc);
      S.ndone += nret;
      S.res -= wave_sum(rl);
      S.nact = N - nret;
      S.min_end = wave_min(me);
      if (S.nact > 0) {
        S.sum_s = (uint32_t)S.nact * (uint32_t)t - (uint32_t)st_g;
        S.min_s = t - st_gmax;
        S.max_s = t - st_gmin;
      } else {
        S.sum_s = 0;
        S.min_s = IDLE;
        S.max_s = -1;
      }
      S.t = tau_end;
      if (++iter > iter_max) {
        failed = true;
        break;
      }
      continue;
    }

    // (5) next event.  A release is an event only if the job could be admitted
    // before anything else happens: ISJL with an idle worker that has nothing
    // planned in Phase TWO, or an empty machine with no plan; LJF at an empty
    // machine; SJF with a free slot; FCFS with a free slot and nothing queued
    // (a queued job left waiting with a slot free is blocked by the KV budget,
    // which changes only at a completion, and it precedes every later arrival).  Otherwise it is folded into the
    // next event (the queue is only read there).
    int tn = S.min_end;
    bool rel_matters;
    if (POL == POL_ISJL) rel_matters = (mode == 0 && free_empty > 0) || (S.nact == 0 && planned == 0);
    else if (POL == POL_LJF) rel_matters = S.nact == 0;
    else if (POL == POL_FCFS)  // a queued head blocks every later arrival in FCFS order
      rel_matters = S.nact < Beff && head == relk;
    else rel_matters = S.nact < Beff;
    // ISJL in FILL (with up to 2 slots per lane) and SJF, with a slot free and
    // jobs queued: the queue's head is held back by the KV budget, which stays
    // fixed until a completion.  An arrival before then is an event only if it
    // precedes that head in the policy's order and fits beside the running jobs;
    // the first such arrival bounds the span.
    const bool blocked_head =
        !PRE && !ROB && qcount > 0 && S.nact > 0 &&
        ((POL == POL_SJF && S.nact < Beff) ||
         (POL == POL_ISJL && K <= 2 && mode == 0 && free_empty > 0 && kv_block));
    if (blocked_head) {
      rel_matters = false;
      const int hr = pool.first();
      int r = relk;
      while (r < n) {
        if ((r >> 6) != chunk) load_chunk(r >> 6);
        const int off = r & (WAVE - 1);
        const bool in = (lane >= off) & (rel_t < tn);
        const bool m = in && rel_r < hr && S.res + plen(W[rel_r]) <= M;
        const uint64_t mm = ballot(m);
        if (mm) {
          tn = min(tn, readlane(rel_t, __builtin_ctzll(mm)));
          break;
        }
        if (ballot((lane >= off) & (rel_t >= tn))) break;  // the rest arrive after the span
        r = (r & ~(WAVE - 1)) + WAVE;
      }
    }
    if (rel_matters && relk < n) {
      if ((relk >> 6) != chunk) load_chunk(relk >> 6);
      tn = min(tn, readlane(rel_t, relk & 63));
    }
    if (POL == POL_ISJL) {
      if (planned > 0 && t_w1 > t) {
        bool w0_wait = readlane(ws_end[0], 0) == IDLE &&
                       ((uint32_t)readlane((int)ws_q[0], 0) & 0xFFFFu) != QNONE;
        if (w0_wait) tn = min(tn, t_w1);
      }
      // (unsigned: any two steps below 2^31 and the one beyond them fit, so an alpha
      // near 2^31, or infinity, leaves tn as it is)
      if (mode == 0 && kv_block)
        tn = (int)min((uint32_t)tn, (uint32_t)S.min_s + (uint32_t)alpha + 1u);
    }
    if (tn == IDLE || tn <= t || ++iter > iter_max) {
      failed = true;
      break;
    }

    // (6) account steps t .. tn-1 (Section 5)
    if (S.nact != 0) account(tn - t);
    S.t = tn;
  }
  if constexpr (DEFER) reduce_lane_sums(lane_sums);

  if (failed) {
    write_marker(a.out, a.out_T, inst, T_INTERNAL, lane);
    return;
  }
  if (lane == 0 && a.out_T) {
    a.out_T[inst] = S.t;
  } else if (lane == 0) {
    fsched_metrics m;
    m.T = S.t;
    m.O = osum;
    m.Q = qsum;
    const int64_t sum_comp = (int64_t)S.sum_start + lsum;
    m.E = (int64_t)acc.E;
    m.C = a.c * (int64_t)S.t + a.tau * (int64_t)(acc.SSM2 >> 1);  // both sums are even
    m.W = a.c * (int64_t)S.t + a.tau * (int64_t)(acc.SM2 >> 1);
    m.sum_completion = sum_comp;
    m.sum_latency = sum_comp - rsum;
    m.sum_extent = (int64_t)acc.X;
    m.busy_steps = acc_busy;
    m.peak_kv = acc.peak;
    m.unfair_steps = acc.unfair;
    m.max_extent = acc_maxext;
    m.max_active = acc_maxact;
    a.out[inst] = m;
  }
}

// Whether a grid of `blocks` blocks of `wpb` waves fits the device at once
// (every block resident from the start); false when the runtime cannot tell.
inline bool resident_at_once(const void* kern, int64_t blocks, int wpb, size_t lds) {
  int per_cu = 0, dev = 0, n_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, wpb * WAVE, lds) != hipSuccess ||
      hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return blocks <= (int64_t)per_cu * n_cu;
}

// The fill sweep serves FCFS and SJF, and ISJL when alpha is at least the length
// limit (A_max, below every length, never exceeds it).  With a finite budget
// ISJL's completions mostly meet the guard one at a time, and its event loop
// runs faster without the sweep's code.
template <int POL, bool ROB = false, bool PRE = false>
hipError_t launch_sim(const SimArgs& a, int K, int NW, int wpb, size_t lds, hipStream_t s) {
  const int64_t blocks = (a.n_inst + wpb - 1) / wpb;
  dim3 grid((unsigned)blocks), block((unsigned)(wpb * WAVE));
  constexpr bool FILL_OK = !ROB && !PRE && POL != POL_LJF;
  constexpr bool FILL_ALWAYS = FILL_OK && POL != POL_ISJL;
  const bool fill = FILL_OK && (FILL_ALWAYS || a.alpha >= (int)LEN_LIMIT);
  // ISJL plan-queue links in HBM scratch (a kernel of its own, up to 8 slots per
  // lane; the fill-sweep kernels run with alpha at least every length, so
  // nothing is planned there)
  const bool qh = POL == POL_ISJL && K <= 8 && !fill && a.qlink != nullptr;
#define FS_LAUNCH(KK, NN, FF, QQ)                                                         \
  if (K == KK && NW == NN && fill == FF && qh == QQ) {                                    \
    if constexpr (KK <= 8) {                                                              \
      if (a.share_simds &&                                                                \
          resident_at_once((const void*)simulate_kernel<POL, KK, NN, ROB, PRE, FF, QQ, true>, \
                           blocks, wpb, lds)) {                                           \
        hipLaunchKernelGGL((simulate_kernel<POL, KK, NN, ROB, PRE, FF, QQ, true>), grid, block, \
                           lds, s, a);                                                    \
        return hipGetLastError();                                                         \
      }                                                                                   \
    }                                                                                     \
    hipLaunchKernelGGL((simulate_kernel<POL, KK, NN, ROB, PRE, FF, QQ>), grid, block, lds, s, \
                       a);                                                                \
    return hipGetLastError();                                                             \
  }
#define FS_LAUNCH_K(KK, FF, QQ) FS_LAUNCH(KK, 1, FF, QQ) FS_LAUNCH(KK, 2, FF, QQ)
  if constexpr (FILL_OK) {
    FS_LAUNCH_K(1, true, false)
    FS_LAUNCH_K(2, true, false)
    FS_LAUNCH_K(4, true, false)
    FS_LAUNCH_K(8, true, false)
    FS_LAUNCH_K(16, true, false)
  }
  if constexpr (!FILL_ALWAYS) {
    FS_LAUNCH_K(1, false, false)
    FS_LAUNCH_K(2, false, false)
    FS_LAUNCH_K(4, false, false)
    FS_LAUNCH_K(8, false, false)
    FS_LAUNCH_K(16, false, false)
  }
  if constexpr (POL == POL_ISJL) {
    FS_LAUNCH_K(1, false, true)
    FS_LAUNCH_K(2, false, true)
    FS_LAUNCH_K(4, false, true)
    FS_LAUNCH_K(8, false, true)
  }
#undef FS_LAUNCH_K
#undef FS_LAUNCH
  return hipErrorInvalidValue;
}

}  // namespace fs
