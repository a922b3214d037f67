// Re-scoring of given schedules (Section 5, profit decomposition; eq. (1) checks):
// one wavefront per instance, two beyond 512 jobs.
//
// The 2n start/end events are sorted in registers as packed keys
//   time << 13 | kind << 12 | index      (kind 0 = end, 1 = start)
// so that at equal times completions come before starts, matching the step
// model (a job ending at t frees its slot for a job starting at t).  Between
// two event times the active set is fixed and the Section 5 terms are summed
// in closed form, as in the simulation kernel; the sweep itself is described
// where it runs.
//
// The sweep is a chain of dependent steps of 64 events, and the sorted events
// and job lengths (20 KB at 2,000 jobs) let 8 instances share a CU's LDS: with
// one wave each, two waves per SIMD, the chain's latency was exposed (VALU busy
// half of the time).  Two waves per instance share its events: each sorts half
// of them (32 keys per lane, which brings the kernel under 128 VGPRs), one
// exchange through LDS and a half-clean merge the halves, and each sweeps its
// half of the sorted events from a state counted from the events before it.
// 65,536 x 2,000: 3.73 -> 3.02 ms (2.80 with the counts from lane masks, the
// doubled sums and the short way through large groups, 2.58 with the sorted keys
// at bank-free places).
#include "dec_common.hpp"
#include "regsort.hpp"
#include "wave.hpp"

namespace fs {

namespace {

constexpr int IDLE32 = 0x7FFFFFFF;

// Totals of the job table that both waves of an instance need.
struct DecShared {
  uint32_t flags, maxlen, tmax, pad;
  unsigned long long osum;
};

// One wave's sums.
struct DecSums {
  uint64_t E, X, SM, SSM, q2;
  int64_t csum, asum;
  uint32_t D, B, U, P;
  int Xm, Am;
  uint32_t v;
};

__device__ inline void dec_marker(fsched_metrics* out, uint32_t* viol, int64_t inst, int64_t code,
                                  uint32_t v, bool writer) {
  if (writer) {
    fsched_metrics m;
    m.T = code;
    m.O = m.Q = m.E = m.C = m.W = 0;
    m.sum_completion = m.sum_latency = m.sum_extent = m.busy_steps = 0;
    m.peak_kv = m.unfair_steps = 0;
    m.max_extent = m.max_active = 0;
    out[inst] = m;
    viol[inst] = v;
  }
}

}  // namespace

// NP2: events, rounded up to a power of two; G: waves per instance (a block of
// its own when there are two).
constexpr int dec_waves(int NP2) { return NP2 > 1024 ? 2 : 1; }

template <int NP2, int G>
__global__ __launch_bounds__(G == 1 ? 256 : WAVE * G)
__attribute__((amdgpu_waves_per_eu(NP2 <= 4096 ? 4 : 2))) void decompose_kernel(DecArgs a) {
  extern __shared__ uint32_t lds_raw[];
  const int wib = threadIdx.x >> 6;
  const int g = G == 1 ? 0 : uni(wib);  // this wave's share of the instance
  const int64_t inst = G == 1 ? (int64_t)blockIdx.x * (blockDim.x >> 6) + wib : (int64_t)blockIdx.x;
  if (inst >= a.n_inst) return;
  const int lane = lane_id();
  const int n = a.n;
  uint32_t* EV = lds_raw + (G == 1 ? (size_t)wib * (size_t)a.wave_words : 0);
  uint16_t* LEN = (uint16_t*)(EV + NP2);  // per job: prompt + output
  DecShared* SH = (DecShared*)(EV + a.wave_words) - 1;
  const int64_t row = inst * (int64_t)n;
  const int32_t* A = a.arrival + row;
  const int32_t* P = a.prompt + row;
  const int32_t* O = a.output + row;
  const int32_t* S0 = a.start + row;
  auto sync = [&]() {
    if constexpr (G == 1) wave_lds_sync();
    else __syncthreads();
  };

  // One pass over the job table: validation, instance totals, the two event
  // keys of every job (end: (s + len, 0, i), start: (s, 1, i); they are only
  // sorted once the table is known to be valid) and the lengths.  The rows are
  // software-pipelined: the loads of row r + PF are issued while row r is
  // processed (clamped indices keep every load in bounds).  Every sum but the
  // arrivals' fits 32 bits per lane in an instance that is scored (at most 64
  // rows, lengths < 2^20, completions < 2^19).
  const int NE = 2 * n;
  if (G > 1) {
    if (threadIdx.x == 0) SH->flags = SH->maxlen = SH->tmax = SH->osum = 0;
    __syncthreads();
  }
  uint32_t bad = 0, neg = 0, early = 0, big = 0, maxlen = 0, tmax = 0;
  uint32_t osum32 = 0, csum32 = 0;
  uint64_t q2 = 0;
  int64_t asum = 0;
  constexpr int PF = 4;
  int pf_a[PF], pf_p[PF], pf_o[PF], pf_s[PF];
#pragma unroll
  for (int d = 0; d < PF; ++d) {
    const int ic = min((d * G + g) * WAVE + lane, n - 1);
    pf_a[d] = A[ic];
    pf_p[d] = P[ic];
    pf_o[d] = O[ic];
    pf_s[d] = S0[ic];
  }
  for (int r0 = g * WAVE; r0 < n; r0 += PF * G * WAVE) {
#pragma unroll
    for (int d = 0; d < PF; ++d) {
      const int i0 = r0 + d * G * WAVE;
      if (i0 >= n) break;
      const int i = i0 + lane;
      const int ar = pf_a[d], p = pf_p[d], o = pf_o[d], s = pf_s[d];
      {
        const int ic = min(i + PF * G * WAVE, n - 1);
        pf_a[d] = A[ic];
        pf_p[d] = P[ic];
        pf_o[d] = O[ic];
        pf_s[d] = S0[ic];
      }
      if (i < n) {
        bad |= (uint32_t)((ar < 0) | (p < 0) | (o < 1));
        const uint32_t len = (uint32_t)p + (uint32_t)o;  // below 2^32 in a valid table
        big |= (uint32_t)(len >= (1u << 20));
        neg |= (uint32_t)(s < 0);
        early |= (uint32_t)(s < ar);
        const uint32_t e = (uint32_t)s + len;
        tmax = max(tmax, e);
        maxlen = max(maxlen, len);
        osum32 += len;
        q2 += (uint64_t)len * (len + 1u);
        csum32 += e;
        asum += ar;
        EV[2 * i] = (e << 13) | (uint32_t)i;
        EV[2 * i + 1] = ((uint32_t)s << 13) | (1u << 12) | (uint32_t)i;
        LEN[i] = (uint16_t)len;
      }
    }
  }
  for (int e = NE + (int)threadIdx.x % (WAVE * G); e < NP2; e += WAVE * G) EV[e] = 0xFFFFFFFFu;
  // completions at or beyond 2^31 (not scored) as the largest signed value
  const uint32_t tcap = min(tmax, 0x7FFFFFFFu), lcap = min(maxlen, 0x7FFFFFFFu);
  uint32_t flags = (ballot(bad != 0) ? 1u : 0u) | (ballot(neg != 0) ? 2u : 0u) |
                   (ballot(early != 0) ? 4u : 0u) | (ballot(big != 0) ? 8u : 0u);
  int maxl = wave_max((int)lcap), tm = wave_max((int)tcap);
  int64_t osum = wave_sum64((int64_t)osum32);
  if constexpr (G > 1) {
    if (lane == 0) {
      atomicOr(&SH->flags, flags);
      atomicMax(&SH->maxlen, (uint32_t)maxl);
      atomicMax(&SH->tmax, (uint32_t)tm);
      atomicAdd(&SH->osum, (unsigned long long)osum);
    }
    __syncthreads();
    flags = uniu(SH->flags);
    maxl = uni((int)SH->maxlen);
    tm = uni((int)SH->tmax);
    osum = uni64((int64_t)SH->osum);
  }
  const bool writer = lane == 0 && g == 0;
  if (flags & 1u) {
    dec_marker(a.out, a.viol, inst, FSCHED_T_INVALID, 0u, writer);
    return;
  }
  if (flags & 2u) {  // a negative start: nothing else is evaluated (bit 16, plus bit 1)
    dec_marker(a.out, a.viol, inst, 0, 16u | 1u, writer);
    return;
  }
  if ((flags & 8u) || (int64_t)tm >= DEC_TIME_LIMIT) {
    dec_marker(a.out, a.viol, inst, FSCHED_T_TOOLARGE, 0u, writer);
    return;
  }
  {
    double cb = (double)a.c * (double)tm + (double)a.tau * (double)osum * (double)maxl;
    double wb = (double)a.c * (double)tm + (double)a.tau * (double)tm * (double)maxl;
    if (cb > 4.0e18 || wb > 4.0e18) {
      dec_marker(a.out, a.viol, inst, FSCHED_T_RANGE, 0u, writer);
      return;
    }
  }
  // a length of 65,536 tokens or more does not fit the 16-bit table: the
  // instance reads its lengths from the job table
  const bool wide = maxl >= 65536;
  auto len_of = [&](uint32_t key) -> int {
    const int i = (int)(key & 0xFFFu);
    return wide ? P[i] + O[i] : (int)LEN[i];
  };

  // The sorted events lie at their bank-free places (swz): in order, the lanes'
  // 32 consecutive events each met in one bank (2.98e8 conflict cycles per launch
  // of 65,536 x 2,000; 2.81 -> 2.61 ms without them).
  // ---- events (keys written above) ---------------------------------------------
  sync();
  {
    constexpr int KS = NP2 / (WAVE * G);  // keys per lane
    uint32_t key[KS];
    uint32_t* mine = EV + g * (KS * WAVE);
#pragma unroll
    for (int k = 0; k < KS; ++k) key[k] = mine[k * WAVE + lane];
    reg_sort_keys<KS, true>(key, lane);
    if constexpr (G == 2) {
      // merge the halves: position p against its mirror NP2 - 1 - p in the other
      // half, the first half keeping the smaller keys, then half-cleaners inside
      // each half.  The halves pass through LDS one row per register.
      __syncthreads();
#pragma unroll
      for (int k = 0; k < KS; ++k) mine[k * WAVE + lane] = key[k];
      __syncthreads();
      const uint32_t* other = EV + (1 - g) * (KS * WAVE);
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const uint32_t x = other[(KS - 1 - k) * WAVE + (WAVE - 1) - lane];
        key[k] = g == 0 ? min(key[k], x) : max(key[k], x);
      }
      reg_sort_halves<KS, true, KS * WAVE / 2>(key, lane);
      __syncthreads();
    } else {
      wave_lds_sync();
    }
#pragma unroll
    for (int k = 0; k < KS; ++k) mine[swz(lane * KS + k)] = key[k];
  }
  sync();

  // ---- sweep ----------------------------------------------------------------
  // 64 sorted events at a time: |S|, the start sum and the reservation sum
  // after each event are prefix scans of the events' deltas.  A group is the
  // events of one time; the span after a group end lasts to the next event
  // time.  The earliest / latest active start after a group end changes only
  // when the group starts jobs or when the last active job holding it ends, so
  // only those group ends are visited one by one: the earliest start is kept
  // with the number of active jobs that started then (nmin; the same for the
  // latest, nmax), and a group end is visited when it has starts or when the
  // ends since the last visit use up nmin or nmax.  A start event is active at
  // time t when its job ends after t; a new earliest (latest) start is searched
  // forward (backward) from the previous one, 64 events per step.  The values
  // in force at every group end are then spread by lane and the span terms of
  // all group ends of the chunk are summed at once.
  const int alpha = a.alpha;
  const int64_t M = a.M;
  const int Bcap = a.B;
  uint32_t v = (flags & 4u) ? 1u : 0u;
  int c_cnt = 0;                       // |S| before the chunk
  // start sum and reservation sum before the chunk: below 4,096 x 2^19, so
  // they (and every partial sum) are exact in 32 bits
  uint32_t c_sum = 0, c_res = 0;
  int min_s = IDLE32, max_s = -1;      // earliest / latest active start
  int nmin = 0, nmax = 0;              // active jobs that started at min_s / max_s
  int pmin = 0, pmax = -1;             // first / last of their start events
  int cnt_last = 0;                    // |S| at the last group end
  int g_nst = 0, gfirst = -1, glast = -1;  // starts of the open group (before this chunk)
  // per lane: E, extent and the doubled largest-footprint sums (C and W take c
  // and tau once at the end) in 64 bits; span lengths, busy and
  // unfair steps (the spans of one lane are disjoint, so each sum stays below
  // 2^19) and peak KV in 32 bits; extent and |S| maxima
  uint64_t lE = 0, lX = 0, lSM2 = 0, lSSM2 = 0;
  uint32_t lD = 0, lB = 0, lU = 0, lP = 0;
  int lXm = 0, lAm = 0;
  bool over = false, lkv = false, lunf = false;
  // idle steps before the first event
  const int t_first = (int)(EV[swz(0)] >> 13);
  const int64_t c0 = a.c * (int64_t)t_first;

  // position of the k-th set bit (k >= 1) of m, which has at least k
  auto kth_bit = [](uint64_t m, int k) -> int {
    int pos = 0;
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
      const uint64_t low = m & ((1ull << w) - 1);
      const int c = __builtin_popcountll(low);
      if (k > c) {
        k -= c;
        m >>= w;
        pos += w;
      } else {
        m = low;
      }
    }
    return pos;
  };
  auto bits_above = [](int d) -> uint64_t {  // lanes > d (d in -1 .. 63)
    return d < 0 ? ~0ull : (d >= 63 ? 0ull : ~((2ull << d) - 1));
  };

  // Span terms of one group end (the span runs to the next event time; the
  // last event has none).  They are added one chunk late, next to the next
  // chunk's scans, which do not depend on them.
  auto span_terms = [&](bool on, int t, int t_next, int cnt_p, uint32_t sum_p, uint32_t res_p,
                        int gmin, int gmax) {
    if (on) {
      // times < 2^19 and |S| <= 4,096: every factor below, and |S| times the
      // span, fit 32 bits, so each product is one 32 x 32 -> 64-bit multiply-add
      const uint32_t D = (uint32_t)(t_next - t);
      lD += D;
      if (cnt_p != 0) {
        const uint32_t s = (uint32_t)cnt_p;
        const uint32_t m0 = (uint32_t)(t - gmin + 1);
        const uint32_t sD = s * D;
        // per step of the span the largest footprint is m0, m0 + 1, ...: its sum
        // is D m0 + D (D - 1) / 2, kept doubled
        const uint32_t m2 = 2u * m0 + D - 1u;
        lSM2 += (uint64_t)D * m2;
        lSSM2 += (uint64_t)sD * m2;
        // sum of (start - earliest start) over the active jobs: < 4,096 x 2^19
        lE += (uint64_t)D * (sum_p - s * (uint32_t)gmin);
        const int ext = gmax - gmin;
        lX += (uint64_t)D * (uint32_t)ext;
        lB += D;
        if (ext > alpha) {
          lU += D;
          lunf = true;
        }
        lXm = max(lXm, ext);
        lAm = max(lAm, cnt_p);
        lP = max(lP, s * (uint32_t)t_next - sum_p);
        if ((Bcap > 0) & (cnt_p > Bcap)) over = true;
        if ((M != 0) & (cnt_p >= 2) & ((int64_t)res_p > M)) lkv = true;
      }
    }
  };
  // the previous chunk's group ends, waiting for their span terms
  bool q_on = false;
  int q_t = 0, q_tn = 0, q_cnt = 0, q_gmin = 0, q_gmax = 0;
  uint32_t q_sum = 0, q_res = 0;
  // This wave's events [p0, p1): with two waves, up to and from the first group
  // that begins in the second half.
  int p0 = 0, p1 = NE;
  if constexpr (G == 2) {
    int bnd = NE;
    for (int q = n; q < NE; q += WAVE) {
      const int e = q + lane;
      const uint64_t m = ballot(e < NE && (EV[swz(e)] >> 13) != (EV[swz(e - 1)] >> 13));
      if (m) {
        bnd = q + __builtin_ctzll(m);
        break;
      }
    }
    if (g == 0) {
      p1 = bnd;
    } else {
      p0 = bnd;
      if (bnd < NE) {
        // the state before it: a job started earlier is active when it ends at
        // that time or later; nmin = nmax = 0 has the first group end search the
        // earliest and latest start, from the first and last such start event
        const int tb = (int)(uniu(EV[swz(bnd)]) >> 13);
        int cnt = 0, first = IDLE32, last = -1;
        uint32_t ss = 0, sr = 0;
        for (int e = lane; e < bnd; e += WAVE) {
          const uint32_t key = EV[swz(e)];
          const int len = len_of(key), t = (int)(key >> 13);
          const bool on = ((key >> 12) & 1u) & (uint32_t)(t + len >= tb);
          cnt += on ? 1 : 0;
          ss += on ? (uint32_t)t : 0u;
          sr += on ? (uint32_t)len : 0u;
          first = min(first, on ? e : IDLE32);
          last = max(last, on ? e : -1);
        }
        c_cnt = cnt_last = wave_sum(cnt);
        c_sum = (uint32_t)wave_sum((int)ss);
        c_res = (uint32_t)wave_sum((int)sr);
        if (c_cnt > 0) {
          pmin = wave_min(first);
          pmax = wave_max(last);
          min_s = (int)(uniu(EV[swz(pmin)]) >> 13);
          max_s = (int)(uniu(EV[swz(pmax)]) >> 13);
        }
      }
    }
  }
  // keys and lengths are loaded one chunk ahead
  uint32_t nkey = p0 + lane < NE ? EV[swz(p0 + lane)] : 0xFFFFFFFFu;
  int nlen = p0 + lane < NE ? len_of(nkey) : 0;

  for (int base = p0; base < p1; base += WAVE) {
    const int p = base + lane;
    const bool valid = p < p1;
    const uint32_t key = nkey;
    const int len = nlen;
    const int pn = p + WAVE;
    nkey = pn < NE ? EV[swz(pn)] : 0xFFFFFFFFu;
    const int t = (int)(key >> 13);
    const bool is_start = valid & (((key >> 12) & 1u) != 0u);
    const bool is_end = valid & (((key >> 12) & 1u) == 0u);
    const int sj = is_start ? t : t - len;  // the job's start
    // within a chunk the deltas sum to less than 64 x 2^20 in magnitude (times
    // < 2^19, lengths < 2^20)
    const int dsum = is_start ? sj : (is_end ? -sj : 0);
    const int dres = is_start ? len : (is_end ? -len : 0);
    nlen = pn < NE ? len_of(nkey) : 0;
    // the next event's time: the lane above, and for the last lane the first
    // key of the next chunk
    int t_next = dpp<DPP_WAVE_SHL1, 0xf, 0xf, false>(t, t);
    const int t_first_next = (int)((uint32_t)readlane((int)nkey, 0) >> 13);
    if (lane == WAVE - 1) t_next = base + WAVE < NE ? t_first_next : t;
    const bool last = p == NE - 1;
    const bool gend = valid & (last | (t_next > t));
    // lane masks, each from one comparison (combined on the scalar unit)
    const int nv = p1 - base;  // valid lanes: 0 .. nv - 1
    const uint64_t vmask = nv >= WAVE ? ~0ull : ((1ull << nv) - 1);
    const uint64_t smask = vmask & ballot((key & 0x1000u) != 0u);
    const uint64_t emask = vmask & ~smask;
    const uint64_t gmask = vmask & (ballot(t_next > t) | ((nv <= WAVE) & (p1 == NE) ? 1ull << (nv - 1) : 0ull));
    uint64_t emin = emask & ballot(sj == min_s);
    uint64_t emax = emask & ballot(sj == max_s);
    span_terms(q_on, q_t, q_tn, q_cnt, q_sum, q_res, q_gmin, q_gmax);
    if (gmask == 0) {
      // the middle of a large group (a batch that starts or ends together: 4 in
      // 10 chunks of the schedules of 512 workers): only the state before the
      // next chunk changes
      q_on = false;
      nmin -= __builtin_popcountll(emin);
      nmax -= __builtin_popcountll(emax);
      if (smask) {
        if (g_nst == 0) gfirst = base + __builtin_ctzll(smask);
        g_nst += __builtin_popcountll(smask);
        glast = base + 63 - __builtin_clzll(smask);
      }
      c_cnt += __builtin_popcountll(smask) - __builtin_popcountll(emask);
      c_sum += (uint32_t)wave_sum(dsum);
      c_res += (uint32_t)wave_sum(dres);
      continue;
    }
    const int cnt_p = c_cnt + mbcnt(smask) - mbcnt(emask) + (is_start ? 1 : (is_end ? -1 : 0));
    const uint32_t sum_p = c_sum + (uint32_t)wave_scan_incl(dsum);
    const uint32_t res_p = c_res + (uint32_t)wave_scan_incl(dres);
    // Common case, with no walk: the active set is never empty at a group end,
    // the earliest start keeps a job through the chunk, and the latest start
    // can only rise: it keeps a job until the chunk's first start (or a group
    // with starts is open from the previous chunk and ends in this one), and no
    // job started in the chunk ends in it while its start is the latest.  Then
    // the earliest start stays, and the latest start at a group end is the
    // later of the one carried in and the latest start time up to it (a prefix
    // max over the chunk; a group's starts come after its ends, so a group end
    // with starts is itself a start and takes its own time).
    int gmin, gmax;
    const int lat = wave_scan_incl_max(is_start ? t : -1);  // latest start time up to the lane
    const int fsl = smask ? __builtin_ctzll(smask) : WAVE;  // first start of the chunk
    const uint64_t pre = fsl >= WAVE ? ~0ull : ((1ull << fsl) - 1);
    const bool open_in = g_nst > 0;  // then the chunk begins with starts of that group
    const bool max_kept = open_in || (nmax > 0 && __builtin_popcountll(emax & pre) < nmax);
    const int g_end = 63 - __builtin_clzll(gmask);  // the chunk's last group end
    const bool fast = min_s != IDLE32 && nmin > 0 && max_kept && !(gmask & ballot(cnt_p == 0)) &&
                      __builtin_popcountll(emin) < nmin && !(emask & ballot(sj == lat));
    if (fast) {
      gmin = min_s;
      gmax = max(max_s, lat);
      nmin -= __builtin_popcountll(emin);
      const uint64_t sg = gmask & smask;  // group ends of groups with starts
      if (sg) {
        // the latest of them: its starts lie after the group end before it,
        // plus those of the previous chunk when it is the open group
        const int gL = 63 - __builtin_clzll(sg);
        const uint64_t below = gmask & ((1ull << gL) - 1);
        const uint64_t rng =
            bits_above(below ? 63 - __builtin_clzll(below) : -1) & (gL == 63 ? ~0ull : ((2ull << gL) - 1));
        max_s = readlane(t, gL);
        nmax = __builtin_popcountll(smask & rng) + (open_in && !below ? g_nst : 0);
        pmax = base + gL;
      } else {
        nmax -= __builtin_popcountll(emax);
      }
      // starts after the chunk's last group end open the next group
      const uint64_t st = smask & bits_above(g_end);
      g_nst = __builtin_popcountll(st);
      if (st) {
        gfirst = base + __builtin_ctzll(st);
        glast = base + 63 - __builtin_clzll(st);
      }
      cnt_last = readlane(cnt_p, g_end);
    } else {
      const int min0 = min_s, max0 = max_s;  // in force before the chunk's first visit
      uint64_t chg = 0;                      // visited group ends
      int vmin = 0, vmax = 0;                // values set there
      int done = -1;                         // lanes <= done are accounted for
      bool open = g_nst > 0;                 // the first group of the chunk began earlier
      while (true) {
        const uint64_t after = bits_above(done);
        const uint64_t ge = gmask & after;
        if (!ge) break;
        // the earliest position after `done` at which something can change
        int x = WAVE;
        if (open || (min_s != IDLE32 && nmin <= 0) || (max_s >= 0 && nmax <= 0)) x = 0;
        const uint64_t sa = smask & after;
        if (sa) x = min(x, __builtin_ctzll(sa));
        if (min_s != IDLE32) {
          const uint64_t ea = emin & after;
          if (__builtin_popcountll(ea) >= nmin && nmin > 0) x = min(x, kth_bit(ea, nmin));
        }
        if (max_s >= 0) {
          const uint64_t ea = emax & after;
          if (__builtin_popcountll(ea) >= nmax && nmax > 0) x = min(x, kth_bit(ea, nmax));
        }
        if (x == WAVE) break;
        const uint64_t gx = ge & ~((1ull << x) - 1);
        if (!gx) break;  // the group ends in the next chunk
        const int gL = __builtin_ctzll(gx);
        const uint64_t rng = after & (gL == 63 ? ~0ull : ((2ull << gL) - 1));
        const int tg = readlane(t, gL);
        const int cnt_g = readlane(cnt_p, gL);
        // |S| before this group: at the previous group end
        const uint64_t gprev = gmask & ((1ull << gL) - 1);
        const int cnt_before = gprev ? readlane(cnt_p, 63 - __builtin_clzll(gprev)) : cnt_last;
        nmin -= __builtin_popcountll(emin & rng);
        nmax -= __builtin_popcountll(emax & rng);
        const uint64_t sr = smask & rng;
        const bool with_open = open && !gprev;
        const int nst = __builtin_popcountll(sr) + (with_open ? g_nst : 0);
        if (nst > 0) {
          const int gf = with_open ? gfirst : base + __builtin_ctzll(sr);
          const int gl = sr ? base + 63 - __builtin_clzll(sr) : glast;
          if (cnt_before == 0) {
            min_s = tg;
            nmin = nst;
            pmin = gf;
          }
          max_s = tg;
          nmax = nst;
          pmax = gl;
        }
        open = open && gprev;  // a group end before gL closed the open group
        if (with_open) open = false;
        const int gpos = base + gL;
        if (cnt_g == 0) {
          min_s = IDLE32;
          max_s = -1;
          nmin = nmax = 0;
        } else {
          if (nmin <= 0) {
            // first active start event at or after pmin; then count the active
            // ones at that time
            int q = max(pmin, 0), found = -1, cnt = 0;
            while (q <= gpos) {
              const int ee = q + lane;
              bool ok = false;
              int st_time = 0;
              if (ee >= 0 && ee <= gpos) {
                const uint32_t kk = EV[swz(ee)];
                st_time = (int)(kk >> 13);
                ok = ((kk >> 12) & 1u) && st_time + len_of(kk) > tg;
              }
              if (found < 0) {
                const uint64_t hm = ballot(ok);
                if (hm) {
                  const int L = __builtin_ctzll(hm);
                  found = q + L;
                  min_s = readlane(st_time, L);
                }
              }
              if (found >= 0) {
                cnt += __builtin_popcountll(ballot(ok & (st_time == min_s)));
                if (ballot((ee >= 0) & (ee <= gpos) & (st_time > min_s))) break;
              }
              q += WAVE;
            }
            pmin = found;
            nmin = cnt;
          }
          if (nmax <= 0) {
            // last active start event at or before pmax; then count the active
            // ones at that time
            int q = pmax, found = -1, cnt = 0;
            while (q >= 0) {
              const int ee = q - lane;
              bool ok = false;
              int st_time = 0;
              if (ee >= 0) {
                const uint32_t kk = EV[swz(ee)];
                st_time = (int)(kk >> 13);
                ok = ((kk >> 12) & 1u) && st_time + len_of(kk) > tg;
              }
              if (found < 0) {
                const uint64_t hm = ballot(ok);
                if (hm) {
                  const int L = __builtin_ctzll(hm);
                  found = q - L;
                  max_s = readlane(st_time, L);
                }
              }
              if (found >= 0) {
                cnt += __builtin_popcountll(ballot(ok & (st_time == max_s)));
                if (ballot((ee >= 0) & (st_time < max_s))) break;
              }
              q -= WAVE;
            }
            pmax = found;
            nmax = cnt;
          }
        }
        chg |= 1ull << gL;
        if (lane == gL) {
          vmin = min_s;
          vmax = max_s;
        }
        emin = emask & ballot(sj == min_s);
        emax = emask & ballot(sj == max_s);
        done = gL;
      }
      // the rest of the chunk: groups with nothing to change, then the open group
      {
        const uint64_t after = bits_above(done);
        nmin -= __builtin_popcountll(emin & after);
        nmax -= __builtin_popcountll(emax & after);
        const uint64_t glast_m = gmask & after;
        if (glast_m) open = false;
        const uint64_t tail = bits_above(g_end) & after;
        const uint64_t st = smask & tail;
        if (st) {
          if (!open) {
            g_nst = 0;
            gfirst = base + __builtin_ctzll(st);
          }
          g_nst += __builtin_popcountll(st);
          glast = base + 63 - __builtin_clzll(st);
          open = true;
        }
        if (!open) g_nst = 0;
        cnt_last = readlane(cnt_p, g_end);
      }
      // earliest / latest start in force at each group end of the chunk
      {
        const uint64_t upto = lane == 63 ? ~0ull : ((2ull << lane) - 1);
        const uint64_t c = chg & upto;
        const int src = c ? 63 - __builtin_clzll(c) : 0;
        const int fmin = __shfl(vmin, src), fmax = __shfl(vmax, src);
        gmin = c ? fmin : min0;
        gmax = c ? fmax : max0;
      }
    }
    q_on = gend & !last;
    q_t = t;
    q_tn = t_next;
    q_cnt = cnt_p;
    q_sum = sum_p;
    q_res = res_p;
    q_gmin = gmin;
    q_gmax = gmax;
    c_cnt = readlane(cnt_p, 63);
    c_sum = (uint32_t)readlane((int)sum_p, 63);
    c_res = (uint32_t)readlane((int)res_p, 63);
  }
  span_terms(q_on, q_t, q_tn, q_cnt, q_sum, q_res, q_gmin, q_gmax);
  DecSums r;
  r.E = (uint64_t)wave_sum64((int64_t)lE);
  r.X = (uint64_t)wave_sum64((int64_t)lX);
  r.SM = (uint64_t)wave_sum64((int64_t)lSM2) >> 1;  // every term is even
  r.SSM = (uint64_t)wave_sum64((int64_t)lSSM2) >> 1;
  r.q2 = (uint64_t)wave_sum64((int64_t)q2);
  r.csum = wave_sum64((int64_t)csum32);
  r.asum = wave_sum64(asum);
  r.D = (uint32_t)wave_sum((int)lD);  // the busy and idle steps after the first event
  r.B = (uint32_t)wave_sum((int)lB);
  r.U = (uint32_t)wave_sum((int)lU);
  r.P = (uint32_t)wave_max((int)lP);  // below 4,096 x 2^19
  r.Xm = wave_max(lXm);
  r.Am = wave_max(lAm);
  if (ballot(lunf)) v |= 8u;
  if (ballot(over)) v |= 2u;
  if (ballot(lkv)) v |= 4u;
  r.v = v;
  if constexpr (G == 2) {
    // the sorted events are no longer read once both waves are here
    __syncthreads();
    DecSums* part = (DecSums*)EV;
    if (g == 1 && lane == 0) *part = r;
    __syncthreads();
    if (g == 1) return;
    const DecSums o = *part;
    r.E += o.E;
    r.X += o.X;
    r.SM += o.SM;
    r.SSM += o.SSM;
    r.q2 += o.q2;
    r.csum += o.csum;
    r.asum += o.asum;
    r.D += o.D;
    r.B += o.B;
    r.U += o.U;
    r.P = max(r.P, o.P);
    r.Xm = max(r.Xm, o.Xm);
    r.Am = max(r.Am, o.Am);
    r.v |= o.v;
  }

  if (lane == 0) {
    fsched_metrics m;
    m.T = tm;
    m.O = osum;
    m.Q = (int64_t)(r.q2 >> 1);  // every term is even
    m.E = (int64_t)r.E;
    m.C = c0 + a.c * (int64_t)r.D + a.tau * (int64_t)r.SSM;
    m.W = c0 + a.c * (int64_t)r.D + a.tau * (int64_t)r.SM;
    m.sum_completion = r.csum;
    m.sum_latency = r.csum - r.asum;
    m.sum_extent = (int64_t)r.X;
    m.busy_steps = r.B;
    m.peak_kv = r.P;
    m.unfair_steps = r.U;
    m.max_extent = r.Xm;
    m.max_active = r.Am;
    a.out[inst] = m;
    a.viol[inst] = r.v;
  }
}

hipError_t launch_decompose(const DecArgs& a0, hipStream_t s) {
  DecArgs a = a0;
  int NP2 = 64;
  while (NP2 < 2 * a.n) NP2 <<= 1;
  // sorted events, then the length of each job (16 bits); two waves also share
  // their instance's totals
  const int G = dec_waves(NP2);
  a.wave_words = NP2 + (a.n + 1) / 2;
  if (G > 1) a.wave_words = ((a.wave_words + 1) & ~1) + (int)sizeof(DecShared) / 4;
  a.wave_words = (a.wave_words + (G > 1 ? 1 : 3)) & ~(G > 1 ? 1 : 3);
  int wpb = G > 1 ? 1 : 4;  // instances per block
  const size_t lds = (size_t)a.wave_words * 4 * wpb;
  const dim3 grid((unsigned)((a.n_inst + wpb - 1) / wpb)), block((unsigned)(wpb * G * WAVE));
#define FS_DEC(E)                                                                            \
  case E: hipLaunchKernelGGL((decompose_kernel<E, dec_waves(E)>), grid, block, lds, s, a); break;
  switch (NP2) {
    FS_DEC(64)
    FS_DEC(128)
    FS_DEC(256)
    FS_DEC(512)
    FS_DEC(1024)
    FS_DEC(2048)
    FS_DEC(4096)
    FS_DEC(8192)
    default: return hipErrorInvalidValue;
  }
#undef FS_DEC
  return hipGetLastError();
}

}  // namespace fs
