// Batched trajectories for small distances (d = 2, 3: at most 2^9 data
// amplitudes).  One persistent launch runs thousands of trajectories with
// their own round counts, depolarizing probabilities and over-rotation
// angles.  The whole data register of a trajectory lives in LDS and a
// workgroup of NW waves runs it (NW = 1: 8 amplitudes per lane; 2: 4; 4: 2);
// a workgroup takes trajectories from a static list (sorted longest-first by
// the host) until the list is exhausted, so every wave reaches the exit.
//
// Per trajectory (set-up): cos/sin of every gate site's angle, the channel
// thresholds j p / 3 and j p / 15, and the noise-free Kraus pair of every
// stabilizer template are tabulated in LDS (angles common to the launch: the
// angle table and Kraus pairs come precomputed and are only copied).
// Per round: one thread per random draw evaluates Philox for the whole round
// (noise locations and measurements), and a wave vote per draw tells which
// noise locations picked a Pauli.
// Per stabilizer circuit (Sec. II.B: one circuit at a time, ancilla measured
// and reset):
//   1. if a location of the circuit drew a Pauli, one lane of wave 0 per
//      block-basis label runs the circuit's ops with the drawn Paulis on the
//      ancilla 2-vector (track_ops); otherwise the tabulated noise-free pair
//      is used;
//   2. each thread loads its amplitudes: the check's first qubits index the
//      thread's registers, its others are the lowest lane bits (their
//      Walsh-Hadamard stages pair lanes through DPP); the thread transforms
//      them to the check basis and accumulates S_0, S_1; wave reductions (and
//      for NW > 1 the waves' totals in wave order) give p1 and the outcome on
//      the device; the thread then applies D_m, transforms back, applies the
//      ZZ layer and 1/sqrt(S_m) and writes the amplitudes back.
// After the last round wave 0 measures the data qubits one by one from the
// highest label down (two-level descent: lane sums, then within one lane).
// TRACE: the instantiation that sv_run_rounds takes, whatever it is asked for:
// it can write the probabilities of the outcomes and the registers before that
// measurement, and keeps the Kraus diagonals in double precision.
#include "kernels_flip.hip"

namespace qec {

static_assert(sizeof(TOp) == 12 && offsetof(TBlock, ops) % 4 == 0,
              "an op is read as three 32-bit words");

constexpr int kSmallBits = 9;
constexpr int kSmallAmps = 1 << kSmallBits;
constexpr int kSmallStab = 8;     // d <= 3
constexpr int kSmallSites = 64;   // gate sites per round, d <= 3
constexpr int kSmallDraws = 128;  // random draws per round, d <= 3

// Per block template, for a trajectory run by NW waves (2^RB amplitudes per
// lane, RB = 3, 2, 1 for NW = 1, 2, 4): where each of a lane's amplitudes and
// each bit of the thread index sit in the register (bit values).  The check's
// first xreg qubits are register bits 0 .. xreg-1, the next xlanes ones are
// thread-index bits 0 .. xlanes-1: local check index of register j on thread
// t = (j & xmask) | (t & (2^xlanes - 1)) << xreg.
struct SmallDesc {
  uint32_t j_off[8];
  uint32_t lane_bit[8];
  uint32_t q_bit[4];
  int n_lane_bits;
  int xlanes;
  uint32_t xmask;
  int xreg;
};

// E: precision of the Kraus diagonals.  Batches keep the register's own; runs
// of sv_run_rounds double, rounded once with the renormalisation (complex64, d
// = 3 with the ZZ layer, registers against 64 bits: 1.5e-7 / 2.6e-7 with float
// diagonals, 1.3e-7 / 2.0e-7 by the register passes, which round once too).
template <typename T, typename E>
struct SmallSlot {
  C2<T> psi[kSmallAmps];
  C2<E> Dc[kSmallStab][2][16];  // noise-free Kraus diagonals per template
  double Wc[kSmallStab][2][16];
  C2<E> D[2][16];               // current block when a Pauli was drawn
  double W[2][16];
  double cs[2 * kSmallSites];   // cos, sin of each site's angle
  double t1[3], t2[15];         // channel thresholds
  double u[kSmallDraws];        // draws of the current round
  uint32_t F;
  int pad;
};

// Angle table and noise-free Kraus pairs of a launch whose over-rotation
// angles are common to every trajectory: computed once on the host and
// copied into each trajectory's slot instead of being rebuilt per trajectory.
struct SmallShared {
  double cs[2 * kSmallSites];
  cd Dc[kSmallStab][2][16];
  double Wc[kSmallStab][2][16];
};

__device__ __forceinline__ uint32_t sslot(uint32_t i) { return i ^ (((i >> 4) ^ (i >> 8)) & 15u); }

// Move of a double between lanes by a DPP pattern (all lanes active).
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_mov_dpp((int)u, CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(u >> 32), CTRL, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

__device__ __forceinline__ double lane_value(double v, int l) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)u, l);
  const int hi = __builtin_amdgcn_readlane((int)(u >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// v of the last lane of the row before (row_bcast:15, rows in row_mask 0xA)
// or of lane 31 (row_bcast:31, rows in 0xC); 0 in the other rows.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_bcast(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, ROWS, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Sums over the 64 lanes of the wave of two values (every lane gets the same
// totals; called with every lane active): lane pairs, quads, eights and rows
// of 16 through DPP; then rows 1 and 3 add the sums of rows 0 and 2, and row
// 3 adds that of rows 0 + 1, so lane 63 holds (S3 + S2) + (S1 + S0), a fixed
// order.  The two reductions' steps are interleaved (two independent chains
// between dependent DPP moves).
__device__ __forceinline__ void wave_total2(double& a, double& b) {
  a += dpp_double<0xB1>(a);
  b += dpp_double<0xB1>(b);
  a += dpp_double<0x4E>(a);
  b += dpp_double<0x4E>(b);
  a += dpp_double<0x141>(a);
  b += dpp_double<0x141>(b);
  a += dpp_double<0x140>(a);
  b += dpp_double<0x140>(b);
  a += dpp_bcast<0x142, 0xA>(a);
  b += dpp_bcast<0x142, 0xA>(b);
  a += dpp_bcast<0x143, 0xC>(a);
  b += dpp_bcast<0x143, 0xC>(b);
  a = lane_value(a, 63);
  b = lane_value(b, 63);
}

// Any set bit in [off, off + len) of the 128-bit mask h1:h0 (len <= 16).
__device__ __forceinline__ bool any_in_window(uint64_t h0, uint64_t h1, int off, int len) {
  uint64_t w;
  if (off >= 64) w = h1 >> (off - 64);
  else if (off == 0) w = h0;
  else w = (h0 >> off) | (h1 << (64 - off));
  return (w & ((1ull << len) - 1)) != 0;
}

// Walsh-Hadamard stage over thread-index bit B (B < 3: lanes of one wave,
// exchanged through DPP) for a thread's NA amplitudes.
template <int B, typename T, int NA>
__device__ __forceinline__ void small_wht_lane_n(C2<T>* v, int tid) {
  const bool upper = (tid >> B) & 1;
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const C2<T> o{lane_partner<B>(v[j].re, upper), lane_partner<B>(v[j].im, upper)};
    v[j] = upper ? C2<T>{o.re - v[j].re, o.im - v[j].im} : C2<T>{v[j].re + o.re, v[j].im + o.im};
  }
}

// Op source of track_ops for a block whose op i, Pauli code and angle sit in
// lane i: the walk reads them with readlane (op index uniform over the wave).
struct LaneOps {
  uint32_t w0, w1, w2;  // the TOp's three words
  uint32_t c;           // Pauli code
  double cos, sin;      // angle of a rotation op
  __device__ __forceinline__ TOp op_here() const {
    const uint32_t w[3] = {w0, w1, w2};
    TOp o;
    __builtin_memcpy(&o, w, sizeof(TOp));
    return o;
  }
  __device__ __forceinline__ TOp op(int i) const {
    const uint32_t w[3] = {(uint32_t)__builtin_amdgcn_readlane((int)w0, i),
                           (uint32_t)__builtin_amdgcn_readlane((int)w1, i),
                           (uint32_t)__builtin_amdgcn_readlane((int)w2, i)};
    TOp o;
    __builtin_memcpy(&o, w, sizeof(TOp));
    return o;
  }
  __device__ __forceinline__ int code(int i) const { return __builtin_amdgcn_readlane((int)c, i); }
  __device__ __forceinline__ cd angle(int i, const TOp&) const {
    return cd{lane_value(cos, i), lane_value(sin, i)};
  }
};

// Tables of a new trajectory: site angles, thresholds, logical |0>.  sites:
// the op of every gate site of the round template (index = site).
// (tid, nl: thread index and threads of the trajectory's workgroup)
template <typename T, typename E>
__device__ void small_setup_tables(SmallSlot<T, E>& S, int tid, int nl, int n, const TOp* sites,
                                   int n_sites, const uint32_t* init_mask, T amp0, const double* eps,
                                   double p, const SmallShared* shared) {
  // cos / sin of every site's angle
  if (shared) {
    for (int k = tid; k < 2 * n_sites; k += nl) S.cs[k] = shared->cs[k];
  } else {
    for (int k = tid; k < n_sites; k += nl) {
      const double beta = op_angle(sites[k], eps);
      S.cs[2 * k] = cos(beta);
      S.cs[2 * k + 1] = sin(beta);
    }
  }
  if (tid < 3) S.t1[tid] = (double)(tid + 1) * p / 3.0;
  if (tid < 15) S.t2[tid] = (double)(tid + 1) * p / 15.0;
  // logical |0>: bit x of init_mask marks the X-stabilizer orbit of 0; thread
  // g writes amplitudes 8 g .. 8 g + 7
  for (int g = tid; g < (1 << (n - 3)); g += nl) {
    const uint32_t bits8 = (init_mask[g >> 2] >> ((g & 3) * 8)) & 0xFFu;
#pragma unroll
    for (int k = 0; k < 8; ++k)
      S.psi[sslot((uint32_t)(g * 8 + k))] = C2<T>{((bits8 >> k) & 1) ? amp0 : (T)0, (T)0};
  }
}

// Noise-free Kraus pair of every template (needs the angle table).
template <typename T, typename E>
__device__ void small_setup_kraus(SmallSlot<T, E>& S, int tid, int nl, int ns, const TBlock* blocks,
                                  int* err, const SmallShared* shared) {
  if (shared) {
    for (int i = tid; i < ns * 32; i += nl) {
      const int s = i >> 5, m = (i >> 4) & 1, x = i & 15;
      const cd d = shared->Dc[s][m][x];
      S.Dc[s][m][x] = C2<E>{(E)d.re, (E)d.im};
      S.Wc[s][m][x] = shared->Wc[s][m][x];
    }
    return;
  }
  const uint8_t none[kMaxOpsBatch] = {};
  for (int i = tid; i < ns * 16; i += nl) {
    const int s = i >> 4, x = i & 15;
    const TBlock& b = blocks[s];
    if (x >= (1 << b.w)) continue;
    cd v0, v1;
    uint32_t cur = 0;
    if (!track_column(b, CsFromTable{S.cs}, none, x, v0, v1, &cur)) atomicOr(err, 1);
    const double norm = b.type == 0 ? 1.0 / (double)(1 << b.w) : 1.0;
    S.Dc[s][0][x] = C2<E>{(E)(v0.re * norm), (E)(v0.im * norm)};
    S.Dc[s][1][x] = C2<E>{(E)(v1.re * norm), (E)(v1.im * norm)};
    S.Wc[s][0][x] = (v0.re * v0.re + v0.im * v0.im) * norm;
    S.Wc[s][1][x] = (v1.re * v1.re + v1.im * v1.im) * norm;
  }
}

// Walsh-Hadamard transform of a thread's NA registers over the check's
// qubits: register bits 0 .. xreg-1, then thread-index bits 0 .. xlanes-1
// (lane pairs through DPP; every lane of the wave takes part).
template <typename T, int NA>
__device__ __forceinline__ void small_wht(C2<T>* v, int xreg, int xlanes, int tid) {
#pragma unroll
  for (int hb = 1; hb < NA; hb <<= 1) {
    if (hb < (1 << xreg)) {
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        if (i & hb) continue;
        const C2<T> a = v[i], b = v[i | hb];
        v[i] = {a.re + b.re, a.im + b.im};
        v[i | hb] = {a.re - b.re, a.im - b.im};
      }
    }
  }
  if (xlanes > 0) small_wht_lane_n<0, T, NA>(v, tid);
  if (xlanes > 1) small_wht_lane_n<1, T, NA>(v, tid);
  if (xlanes > 2) small_wht_lane_n<2, T, NA>(v, tid);
}

// NW waves (64 NW threads) run one trajectory at a time; lane bits and the
// wave index together form the thread-index bits of the register layout.
template <typename T, int NW, bool TRACE>
__global__ __launch_bounds__(64 * NW) void k_batch_small(
    const TBlock* __restrict__ blocks, const SmallDesc* __restrict__ sdesc, int ns, int n,
    int draws_round, const JobConst* __restrict__ jc, const uint64_t* __restrict__ tseed,
    const uint64_t* __restrict__ tstream,
    const int* __restrict__ order, int n_traj, const int* __restrict__ rounds,
    const double* __restrict__ pvec, const double* __restrict__ eps, int eps_stride,
    uint8_t* __restrict__ rec, int max_rounds, uint8_t* __restrict__ bits, int* __restrict__ err,
    const TOp* __restrict__ sites, int n_sites, const SmallShared* __restrict__ shared,
    const uint32_t* __restrict__ init_mask, const uint8_t* __restrict__ draw_kind, double* __restrict__ p1_out,
    C2<T>* __restrict__ regs_out) {
  static_assert(NW == 1 || NW == 2 || NW == 4, "one, two or four waves per trajectory");
  constexpr int NL = 64 * NW;                       // threads of a trajectory
  constexpr int NA = NW == 1 ? 8 : NW == 2 ? 4 : 2;  // amplitudes per thread
  constexpr int DR = (kSmallDraws + NL - 1) / NL;   // draws per thread and round
  using E = std::conditional_t<TRACE, double, T>;
  __shared__ SmallSlot<T, E> S;
  // ZZ phases are read per amplitude: keep them in LDS (the round template
  // stays in global memory: more LDS per workgroup would cost occupancy)
  __shared__ C2<T> lzz[kSmallBits * 2 + 1];
  __shared__ uint64_t lhits[2];       // noise hits of the round (draws 0..63, 64..127)
  __shared__ double lsum[2][NW];      // per-wave S_0, S_1 of the current circuit
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i <= jc->n_edges && i <= 2 * kSmallBits; i += NL)
    lzz[i] = C2<T>{(T)jc->zz[2 * i], (T)jc->zz[2 * i + 1]};
  const int use_zz = jc->use_zz, zd = jc->d;
  const uint32_t hmask = jc->hmask, vmask = jc->vmask;
  const T amp0 = (T)jc->amp0;
  const int groups = 1 << (n - 3);
  __syncthreads();

  for (int qi = blockIdx.x; qi < n_traj; qi += gridDim.x) {
    const int t = order[qi];
    const int R = rounds[t];
    const double p = pvec[t];
    const uint64_t tg = tstream[t], seed = tseed[t];  // draw stream of this trajectory
    small_setup_tables(S, tid, NL, n, sites, n_sites, init_mask, amp0, eps + (size_t)t * eps_stride, p,
                       shared);
    __syncthreads();
    small_setup_kraus(S, tid, NL, ns, blocks, err, shared);
    __syncthreads();
    for (int r = 0; r < R; ++r) {
      // every draw of the round; hit: a noise location that picked a Pauli
#pragma unroll
      for (int c = 0; c < DR; ++c) {
        const int k = tid + NL * c;
        bool hit = false;
        if (k < draws_round) {
          const double u = uniform(seed, tg, (uint64_t)r * (uint64_t)draws_round + (uint64_t)k);
          S.u[k] = u;
          const int kind = draw_kind[k];
          hit = kind < 2 && u < (kind ? S.t2[14] : S.t1[2]);
        }
        const uint64_t h = __ballot(hit);
        const int chunk = wave + NW * c;
        if (lane == 0 && chunk < 2) lhits[chunk] = h;
      }
      __syncthreads();
      const uint64_t hits0 = lhits[0], hits1 = lhits[1];
      for (int s = 0; s < ns; ++s) {
        const TBlock& b = blocks[s];
        const SmallDesc& sd = sdesc[s];
        const int off = b.draw_off, nnoise = b.n_draws - 1;
        // noise draws off .. off + nnoise - 1 (at most 15, within 128)
        const bool noisy = any_in_window(hits0, hits1, off, nnoise);
        // 1. Kraus pair of this block instance
        const int nx = 1 << b.w;
        if (noisy) {
          // (wave 0) op i of the block, its Pauli code and its angle's
          // (cos, sin) go to lane i (one load and one table lookup in
          // parallel); the lanes of the block-basis labels then walk the
          // ops reading them with readlane
          if (wave == 0) {
            const int nops = b.n_ops;
            LaneOps lo{};
            if (lane < nops) {
              const uint32_t* w = reinterpret_cast<const uint32_t*>(&b.ops[lane]);
              lo.w0 = w[0];
              lo.w1 = w[1];
              lo.w2 = w[2];
              const TOp op = lo.op_here();
              int c = 0;
              if (op.draw >= 0) {
                const double u = S.u[off + op.draw];
                // first threshold above u (thresholds increase with j)
                if (op.kind == OP_N1_ANC || op.kind == OP_N1_DATA) {
                  if (u < S.t1[2]) c = 1 + (u >= S.t1[0]) + (u >= S.t1[1]);
                } else if (u < S.t2[14]) {
                  c = 1;
#pragma unroll
                  for (int j = 0; j < 14; ++j) c += u >= S.t2[j];
                }
              }
              lo.c = (uint32_t)c;
              if (is_rotation(op.kind)) {
                lo.cos = S.cs[2 * op.site];
                lo.sin = S.cs[2 * op.site + 1];
              }
            }
            if (lane < nx) {
              cd v0, v1;
              uint32_t cur = 0;
              if (!track_ops(b.type == 0, nops, lo, lane, v0, v1, &cur)) atomicOr(err, 1);
              const double norm = b.type == 0 ? 1.0 / (double)nx : 1.0;
              S.D[0][lane] = C2<E>{(E)(v0.re * norm), (E)(v0.im * norm)};
              S.D[1][lane] = C2<E>{(E)(v1.re * norm), (E)(v1.im * norm)};
              S.W[0][lane] = (v0.re * v0.re + v0.im * v0.im) * norm;
              S.W[1][lane] = (v1.re * v1.re + v1.im * v1.im) * norm;
              if (lane == 0) S.F = cur;  // label 0 maps to F
            }
          }
          __syncthreads();
        }
        const C2<E>(*D)[16] = noisy ? S.D : S.Dc[s];
        const double(*W)[16] = noisy ? S.W : S.Wc[s];
        const uint32_t F = noisy ? S.F : 0u;
        // 2. measure and apply
        const bool g_on = tid < (1 << sd.n_lane_bits);
        uint32_t lb = 0;
        for (int i = 0; i < sd.n_lane_bits; ++i)
          if ((tid >> i) & 1) lb |= sd.lane_bit[i];
        const uint32_t xm = sd.xmask;
        const int xreg = sd.xreg, xlanes = sd.xlanes;
        const uint32_t xhi = (uint32_t)(tid & ((1 << xlanes) - 1)) << xreg;  // local bits from the thread
        C2<T> v[NA];
#pragma unroll
        for (int j = 0; j < NA; ++j) v[j] = C2<T>{(T)0, (T)0};
        double s0 = 0.0, s1 = 0.0;
        const bool xb = b.type == 0;
        if (g_on) {
#pragma unroll
          for (int j = 0; j < NA; ++j) v[j] = S.psi[sslot(lb | sd.j_off[j])];
        }
        if (xb) small_wht<T, NA>(v, xreg, xlanes, tid);  // every lane joins the lane exchange
        if (g_on) {
#pragma unroll
          for (int j = 0; j < NA; ++j) {
            const uint32_t x = ((uint32_t)j & xm) | xhi;
            const double re = (double)v[j].re, im = (double)v[j].im, a2 = re * re + im * im;
            s0 += W[0][x] * a2;
            s1 += W[1][x] * a2;
          }
        }
        wave_total2(s0, s1);
        if constexpr (NW > 1) {
          // the waves' totals in wave order (the same sum on every wave)
          if (lane == 0) {
            lsum[0][wave] = s0;
            lsum[1][wave] = s1;
          }
          __syncthreads();
          s0 = lsum[0][0];
          s1 = lsum[1][0];
#pragma unroll
          for (int w = 1; w < NW; ++w) {
            s0 += lsum[0][w];
            s1 += lsum[1][w];
          }
        }
        // both renormalisations alongside p1 (the kept one has S_m > 0)
        const double r0 = rsqrt(s0), r1 = rsqrt(s1);
        const double p1 = clamp_p1(s1 / (s0 + s1));
        const int m = (S.u[off + nnoise] < p1) ? 1 : 0;
        if (tid == 0) rec[((size_t)t * max_rounds + r) * ns + s] = (uint8_t)m;
        if (TRACE && p1_out && tid == 0) p1_out[((size_t)t * max_rounds + r) * ns + s] = p1;
        const double scale = m ? r1 : r0;
        if (g_on) {
#pragma unroll
          for (int j = 0; j < NA; ++j) {
            const uint32_t x = ((uint32_t)j & xm) | xhi;
            // (TRACE: the renormalisation with the factor, one rounding less)
            const C2<E> e = D[m][x];
            v[j] = TRACE ? mulc(v[j], (T)(e.re * scale), (T)(e.im * scale)) : mulc(v[j], (T)e.re, (T)e.im);
          }
        }
        if (xb) small_wht<T, NA>(v, xreg, xlanes, tid);
        if (g_on) {
          uint32_t fo = 0;
          if (!xb)
            for (int l = 0; l < b.w; ++l)
              if ((F >> l) & 1) fo |= sd.q_bit[l];
          const T sc = (T)scale;
#pragma unroll
          for (int j = 0; j < NA; ++j) {
            C2<T> o = v[j];
            const uint32_t x = ((uint32_t)j & xm) | xhi;
            if (xb && (__popc(x & F) & 1)) o = {-o.re, -o.im};
            const uint32_t g = (lb | sd.j_off[j]) ^ fo;
            if (use_zz) {
              const int k = __popc((g ^ (g >> 1)) & hmask) + __popc((g ^ (g >> zd)) & vmask);
              o = mulc(o, lzz[k].re, lzz[k].im);
            }
            if (!TRACE) {
              o.re *= sc;
              o.im *= sc;
            }
            S.psi[sslot(g)] = o;
          }
        }
        __syncthreads();
      }
    }
    if (TRACE && regs_out)
      for (int i = tid; i < (1 << n); i += NL) regs_out[((size_t)t << n) + i] = S.psi[sslot((uint32_t)i)];
    // final Z measurement of the data register, highest label first, by wave
    // 0: lane l holds amplitudes 8 l .. 8 l + 7
    if (wave == 0) {
      const bool g_on = lane < groups;
      double L = 0.0;
      if (g_on) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const C2<T> a = S.psi[sslot((uint32_t)(lane * 8 + k))];
          L += (double)a.re * (double)a.re + (double)a.im * (double)a.im;
        }
      }
      const uint64_t kf = (uint64_t)R * (uint64_t)draws_round;
      const double uf = lane < n ? uniform(seed, tg, kf + (uint64_t)lane) : 0.0;
      int lo = 0, size = groups, level = 0;
      for (; level < n - 3; ++level) {
        const int half = size >> 1;
        const bool in0 = lane >= lo && lane < lo + half;
        const bool in1 = lane >= lo + half && lane < lo + size;
        double S0 = in0 ? L : 0.0, S1 = in1 ? L : 0.0;
        wave_total2(S0, S1);
        const double pf = clamp_p1(S1 / (S0 + S1));
        const double u = lane_value(uf, level);
        const int bit = (u < pf) ? 1 : 0;
        if (lane == 0) bits[(size_t)t * n + (n - 1 - level)] = (uint8_t)bit;
        if (bit) lo += half;
        size = half;
      }
      // within the selected lane's 8: every lane reads the same amplitudes
      int lo2 = 0, size2 = 8;
      for (; level < n; ++level) {
        const int half = size2 >> 1;
        double S0 = 0.0, S1 = 0.0;
        for (int k = 0; k < size2; ++k) {
          const C2<T> a = S.psi[sslot((uint32_t)(lo * 8 + lo2 + k))];
          const double w = (double)a.re * (double)a.re + (double)a.im * (double)a.im;
          if (k < half) S0 += w; else S1 += w;
        }
        const double pf = clamp_p1(S1 / (S0 + S1));
        const double u = lane_value(uf, level);
        const int bit = (u < pf) ? 1 : 0;
        if (lane == 0) bits[(size_t)t * n + (n - 1 - level)] = (uint8_t)bit;
        if (bit) lo2 += half;
        size2 = half;
      }
    }
    __syncthreads();  // the slot is rewritten by the next trajectory
  }
}

// ------------------------------------------- d = 3 without the data ZZ layer --
// The register of a d = 3 trajectory (512 amplitudes) stays in one wave's
// registers for the whole trajectory, eight amplitudes a lane, and each round
// goes through two chains of four checks: the X checks in the Hadamard basis,
// the Z checks in the computational one (see k_flip), with a Walsh-Hadamard
// transform of all nine qubits between them.  k_batch_small's circuits are a
// dependent chain of about 2.5 us each, eight a round; here a chain's 16 sums
// come out of one reduction, and its four outcomes out of four divisions side
// by side: every lane forms the conditional probabilities of its own outcome
// prefix, a vote per member compares them with the member's draw, and the
// drawn outcomes are read off the votes one after another.  Bound by vector
// instructions (some 2000 a round, 2500 to set a trajectory up): 65 536 ragged
// complex64 trajectories 4.74 -> 1.60 ms, 1000 complex128 textbook ones of
// three rounds 78 -> 33 us.  TRACE as for k_batch_small (an outcome's
// p1 is in the lane of its prefix), but with the register's own precision for
// the diagonals: one chain's rounding replaces four circuits' (complex64
// registers against 64 bits 9.0e-8, by the passes 9.8e-8; double ones 7.1e-8,
// and 65 536 trajectories of five rounds 1.15 -> 1.67 ms).
//
// Lane bits are qubits 1, 3, 4, 5, 6, 7; register bits the corners 0, 2 and 8,
// each of which belongs to one X check and one Z check only, so that those
// checks' weights contract the eight norms of a lane directly.
constexpr int kFlipSmallSites = 56, kFlipSmallDraws = 72;  // per round, cross-resonance circuit
constexpr int kFlipSmallCols = 80;  // four checks of 16 labels, four of 4
struct FlipSmallDesc {
  uint32_t lane_pack[6];   // lane bit k: its bit in the packed local indices of the eight checks (4 bits each)
  uint32_t reg_bit[2][3];  // register bit k: its bit in its owner's local index (X, Z)
  uint32_t q[8][4];        // global bits of each check's qubits
  uint32_t parity[4];      // X checks: global masks (the initial state's conditions)
  int w[8];
  int col[8];              // first column of each check in the packed Kraus tables
  int col_of[kFlipSmallCols];  // (check << 4 | label) of each column
  int meas[8];             // the measurement draw of each check within the round
};
constexpr int kFlipLaneQubit[6] = {1, 3, 4, 5, 6, 7};
constexpr int kFlipRegQubit[3] = {0, 2, 8};
// owners of the register bits among the four checks of a type, and the one
// check without a corner (Table I order at d = 3: X {0,1} {1,2,4,5} {3,4,6,7}
// {7,8}, Z {3,6} {0,1,3,4} {4,5,7,8} {2,5})
constexpr int kFlipOwnX[4] = {0, 1, 3, 2};
constexpr int kFlipOwnZ[4] = {1, 3, 2, 0};

// (More waves hide more of the dependent chain: 20 000 ragged complex64
// trajectories 0.95 / 0.62 / 0.54 / 0.50 ms with 4 / 8 / 12 / 16 waves a
// compute unit, so the kernel is held to 128 registers, complex128 to 168.)
template <typename T>
struct FlipSmallSlot {
  C2<T> D[2][2][kFlipSmallCols];  // Kraus diagonals by outcome: noise-free, with this round's Paulis
  double W[2][2][kFlipSmallCols];
  double cs[2 * kFlipSmallSites];
  double t1[3], t2[15];
  double u[kFlipSmallDraws];
  uint32_t F[8];
};

// Value of lane l ^ (1 << B), B = 0..3.
template <int B, typename T>
__device__ __forceinline__ T small_xor(T v) {
  if constexpr (B < 3) {
    return lane_xor<B>(v);
  } else {
    return dpp_mv<0x128>(v);  // row_ror:8 within the row of 16
  }
}

// Walsh-Hadamard transform (not normalised) of the wave's 512 amplitudes.
template <typename T>
__device__ __forceinline__ void small_wht_all(C2<T>* v, int lane) {
#pragma unroll
  for (int h = 1; h < 8; h <<= 1)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i & h) continue;
      const C2<T> a = v[i], b = v[i | h];
      v[i] = {a.re + b.re, a.im + b.im};
      v[i | h] = {a.re - b.re, a.im - b.im};
    }
  auto stage = [&](auto bv) {
    constexpr int B = decltype(bv)::value;
    const T sg = ((lane >> B) & 1) ? (T)-1 : (T)1;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const T re = small_xor<B>(v[j].re), im = small_xor<B>(v[j].im);
      v[j].re = fma(v[j].re, sg, re);
      v[j].im = fma(v[j].im, sg, im);
    }
  };
  stage(std::integral_constant<int, 0>{});
  stage(std::integral_constant<int, 1>{});
  stage(std::integral_constant<int, 2>{});
  stage(std::integral_constant<int, 3>{});
  // lane bits 4 and 5: changed places with register bit 2, and back
  auto swapped = [&](auto b32) {
    constexpr bool B32 = decltype(b32)::value;
#pragma unroll
    for (int j = 0; j < 4; ++j) swap_c2<T, B32>(v[j], v[j + 4]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const C2<T> a = v[j], b = v[j + 4];
      v[j] = {a.re + b.re, a.im + b.im};
      v[j + 4] = {a.re - b.re, a.im - b.im};
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) swap_c2<T, B32>(v[j], v[j + 4]);
  };
  swapped(std::integral_constant<bool, false>{});
  swapped(std::integral_constant<bool, true>{});
}

// a + (a of the other half of the wave / the other row of its pair).
template <bool B32>
__device__ __forceinline__ double pair_sum(double a) {
  double b = a;
  swap_d<B32>(a, b);
  return a + b;
}

template <typename T, bool TRACE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 3 : 4))) void k_batch_flip(
    const TBlock* __restrict__ blocks, const FlipSmallDesc* __restrict__ fd, int draws_round,
    const uint64_t* __restrict__ tseed, const uint64_t* __restrict__ tstream, const int* __restrict__ order, int n_traj,
    const int* __restrict__ rounds, const double* __restrict__ pvec, const double* __restrict__ eps, int eps_stride,
    uint8_t* __restrict__ rec, int max_rounds, uint8_t* __restrict__ bits, int* __restrict__ err,
    const TOp* __restrict__ sites, int n_sites, const SmallShared* __restrict__ shared,
    const uint8_t* __restrict__ draw_kind, double* __restrict__ p1_out, C2<T>* __restrict__ regs_out) {
  constexpr int kN = 9, kStab = 8;
  __shared__ FlipSmallSlot<T> S;
  __shared__ uint32_t ops[kStab][kMaxOpsBatch][3];  // the round template's ops
  const int lane = threadIdx.x;
  for (int i = lane; i < kStab * kMaxOpsBatch; i += 64) {
    const TBlock& b = blocks[i / kMaxOpsBatch];
    if (i % kMaxOpsBatch < b.n_ops)
      for (int k = 0; k < 3; ++k)
        ops[i / kMaxOpsBatch][i % kMaxOpsBatch][k] = reinterpret_cast<const uint32_t*>(&b.ops[i % kMaxOpsBatch])[k];
  }
  // this lane's packed local indices and global bits
  uint32_t pl = 0, gl = 0;
#pragma unroll
  for (int k = 0; k < 6; ++k)
    if ((lane >> k) & 1) {
      pl ^= fd->lane_pack[k];
      gl |= 1u << kFlipLaneQubit[k];
    }
  constexpr double kHalf9 = 0.044194173824159216;  // 2^(-9/2)
  __syncthreads();

  for (int qi = blockIdx.x; qi < n_traj; qi += gridDim.x) {
    const int t = order[qi];
    const int R = rounds[t];
    const double p = pvec[t];
    const uint64_t tg = tstream[t], seed = tseed[t];
    // tables: angles, thresholds, noise-free Kraus pairs
    if (shared) {
      for (int k = lane; k < 2 * n_sites; k += 64) S.cs[k] = shared->cs[k];
      for (int i = lane; i < kFlipSmallCols; i += 64) {
        const int s = fd->col_of[i] >> 4, x = fd->col_of[i] & 15;
        const double f = s < 4 ? (double)(1 << fd->w[s]) : 1.0;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const cd d = shared->Dc[s][m][x];
          S.D[0][m][i] = C2<T>{(T)(d.re * f), (T)(d.im * f)};
          S.W[0][m][i] = shared->Wc[s][m][x] * f;
        }
      }
    } else {
      for (int k = lane; k < n_sites; k += 64) {
        const double beta = op_angle(sites[k], eps + (size_t)t * eps_stride);
        S.cs[2 * k] = cos(beta);
        S.cs[2 * k + 1] = sin(beta);
      }
    }
    if (lane < 3) S.t1[lane] = (double)(lane + 1) * p / 3.0;
    if (lane < 15) S.t2[lane] = (double)(lane + 1) * p / 15.0;
    __syncthreads();
    // column x of check s's Kraus pair (table sel), the op source given
    auto column = [&](const auto& src, int sel, int s, int n_ops, int x) {
      cd v0, v1;
      uint32_t cur = 0;
      if (!track_ops(s < 4, n_ops, src, x, v0, v1, &cur)) atomicOr(err, 1);
      const int c = fd->col[s] + x;
      S.D[sel][0][c] = C2<T>{(T)v0.re, (T)v0.im};
      S.D[sel][1][c] = C2<T>{(T)v1.re, (T)v1.im};
      S.W[sel][0][c] = v0.re * v0.re + v0.im * v0.im;
      S.W[sel][1][c] = v1.re * v1.re + v1.im * v1.im;
      if (x == 0) S.F[s] = cur;
    };
    if (!shared) {
      struct LdsOps {
        const uint32_t (*w)[3];
        const double* cs;
        __device__ __forceinline__ TOp op(int i) const {
          TOp o;
          __builtin_memcpy(&o, w[i], sizeof(TOp));
          return o;
        }
        __device__ __forceinline__ int code(int) const { return 0; }
        __device__ __forceinline__ cd angle(int, const TOp& o) const { return cd{cs[2 * o.site], cs[2 * o.site + 1]}; }
      };
      for (int i = lane; i < kFlipSmallCols; i += 64) {
        const int s = fd->col_of[i] >> 4;
        column(LdsOps{ops[s], S.cs}, 0, s, blocks[s].n_ops, fd->col_of[i] & 15);
      }
    }
    // logical |0> in the Hadamard basis: even parity on every X check
    C2<T> v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      uint32_t g = gl;
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if ((j >> k) & 1) g |= 1u << kFlipRegQubit[k];
      bool on = true;
#pragma unroll
      for (int i = 0; i < 4; ++i) on = on && !(__popc(g & fd->parity[i]) & 1);
      v[j] = C2<T>{on ? (T)0.17677669529663688 : (T)0, (T)0};  // 2^(-5/2)
    }
    uint32_t phz = 0, phx = 0;  // frames (see FlipPass)
    int neg = 0;                // and the sign (TRACE)
    for (int r = 0; r < R; ++r) {
      // the round's draws and the noise locations that picked a Pauli
      uint64_t hits[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int k = lane + 64 * c;
        bool hit = false;
        if (k < draws_round) {
          const double u = uniform(seed, tg, (uint64_t)r * (uint64_t)draws_round + (uint64_t)k);
          S.u[k] = u;
          const int kind = draw_kind[k];
          hit = kind < 2 && u < (kind ? S.t2[14] : S.t1[2]);
        }
        hits[c] = __ballot(hit);
      }
      __syncthreads();
      uint32_t noisy = 0;  // checks with a Pauli this round
      if (hits[0] | hits[1])
        for (int s = 0; s < kStab; ++s) {
          const TBlock& b = blocks[s];
          if (!any_in_window(hits[0], hits[1], b.draw_off, b.n_draws - 1)) continue;
          noisy |= 1u << s;
          // op i of the check, its Pauli code and its angle go to lane i; the
          // lanes of the labels walk the ops with readlane
          LaneOps lo{};
          if (lane < b.n_ops) {
            lo.w0 = ops[s][lane][0];
            lo.w1 = ops[s][lane][1];
            lo.w2 = ops[s][lane][2];
            const TOp op = lo.op_here();
            int c = 0;
            if (op.draw >= 0) {
              const double u = S.u[b.draw_off + op.draw];
              if (op.kind == OP_N1_ANC || op.kind == OP_N1_DATA) {
                if (u < S.t1[2]) c = 1 + (u >= S.t1[0]) + (u >= S.t1[1]);
              } else if (u < S.t2[14]) {
                c = 1;
#pragma unroll
                for (int j = 0; j < 14; ++j) c += u >= S.t2[j];
              }
            }
            lo.c = (uint32_t)c;
            if (is_rotation(op.kind)) {
              lo.cos = S.cs[2 * op.site];
              lo.sin = S.cs[2 * op.site + 1];
            }
          }
          if (lane < (1 << b.w)) column(lo, 1, s, b.n_ops, lane);
        }
      __syncthreads();
      // one chain: the four checks c0 .. c0 + 3 of a type, owners of the
      // register bits O0, O1, O2 and the check without one, O3
      auto chain = [&](auto c0v, auto o0, auto o1, auto o2, auto o3) {
        constexpr int C0 = decltype(c0v)::value;
        constexpr bool X = C0 == 0;
        constexpr int O[4] = {decltype(o0)::value, decltype(o1)::value, decltype(o2)::value, decltype(o3)::value};
        // frame: each member's local offset, then its XOR pattern
        uint32_t& ph = X ? phx : phz;
        uint32_t off = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (ph) off |= gather_loc(ph, fd->q[C0 + i], fd->w[C0 + i]) << (4 * i);
          if ((noisy >> (C0 + i)) & 1) {
            const uint32_t G = scatter_loc(S.F[C0 + i], fd->q[C0 + i], fd->w[C0 + i]);
            if (TRACE && X) neg ^= __popc(G & phz) & 1;
            ph ^= G;
          }
        }
        ph = (uint32_t)__builtin_amdgcn_readfirstlane((int)ph);
        const uint32_t xl = (X ? pl & 0xFFFFu : pl >> 16) ^ off;
        auto column_of = [&](int i) { return (uint32_t)fd->col[C0 + i] + ((xl >> (4 * i)) & 15u); };
        auto sel = [&](int i) { return (noisy >> (C0 + i)) & 1; };
        // (labels of a check start at a multiple of four or sixteen columns:
        // a label's bit is the column's)
        // the norms against the owners' weights, one register bit at a time
        double z[8];
        {
          double a[8];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const double re = (double)v[j].re, im = (double)v[j].im;
            a[j] = fma(re, re, im * im);
          }
          double w[3][2][2];  // [register bit][outcome][bit value]
#pragma unroll
          for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
              for (int b = 0; b < 2; ++b)
                w[k][h][b] = S.W[sel(O[k])][h][column_of(O[k]) ^ (b ? fd->reg_bit[X ? 0 : 1][k] : 0u)];
          double y[8];
#pragma unroll
          for (int j = 0; j < 8; j += 2)  // register bit 0 -> outcome of O0
#pragma unroll
            for (int h = 0; h < 2; ++h) y[j + h] = fma(w[0][h][0], a[j], w[0][h][1] * a[j + 1]);
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            if (j & 2) continue;
#pragma unroll
            for (int h = 0; h < 2; ++h) a[j + 2 * h] = fma(w[1][h][0], y[j], w[1][h][1] * y[j + 2]);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) z[j + 4 * h] = fma(w[2][h][0], a[j], w[2][h][1] * a[j + 4]);
        }
        double m3;
        {
          const double u0 = S.W[sel(O[3])][0][column_of(O[3])];
          const double u1 = S.W[sel(O[3])][1][column_of(O[3])];
          double s[16];  // outcome string: bit i is member i's
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            constexpr int B0 = 1 << O[0], B1 = 1 << O[1], B2 = 1 << O[2], B3 = 1 << O[3];
            const int h = (j & 1 ? B0 : 0) | (j & 2 ? B1 : 0) | (j & 4 ? B2 : 0);
            s[h] = z[j] * u0;
            s[h | B3] = z[j] * u1;
          }
          m3 = wave_reduce16(s);  // lane l: string (l >> 2) & 15
        }
        // sums over the later members' outcomes, for every prefix
        const double m2 = pair_sum<true>(m3);
        const double m1 = pair_sum<false>(m2);
        const double m0 = m1 + small_xor<3>(m1);
        const double mt = m0 + small_xor<2>(m0);
        // p1 of each member after this lane's prefix (lanes whose bit is set)
        double p1[4] = {clamp_p1(m0 / mt), clamp_p1(m1 / m0), clamp_p1(m2 / m1), clamp_p1(m3 / m2)};
        uint32_t h = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint64_t vote = __ballot(S.u[fd->meas[C0 + i]] < p1[i]);
          if (TRACE && p1_out && lane == (int)(4 * (h | (1u << i))))
            p1_out[((size_t)t * max_rounds + r) * kStab + C0 + i] = p1[i];
          h |= (uint32_t)((vote >> (4 * (h | (1u << i)))) & 1) << i;
        }
        const double Sm = lane_value(m3, (int)(4 * h));
        if (lane == 0) {
          uint8_t* o = rec + ((size_t)t * max_rounds + r) * kStab + C0;
#pragma unroll
          for (int i = 0; i < 4; ++i) o[i] = (uint8_t)((h >> i) & 1);
        }
        // apply the outcomes (and 1/sqrt(S_m), and the next transform's
        // normalisation)
        const double scale = rsqrt(Sm) * (X || r + 1 < R ? kHalf9 : 1.0);
        C2<T> f[3][2];
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
          for (int b = 0; b < 2; ++b)
            f[k][b] = S.D[sel(O[k])][(h >> O[k]) & 1][column_of(O[k]) ^ (b ? fd->reg_bit[X ? 0 : 1][k] : 0u)];
        C2<T> f3 = S.D[sel(O[3])][(h >> O[3]) & 1][column_of(O[3])];
        f3 = C2<T>{(T)((double)f3.re * scale), (T)((double)f3.im * scale)};
#pragma unroll
        for (int b = 0; b < 2; ++b) f[2][b] = mulc(f[2][b], f3.re, f3.im);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const C2<T> e = mulc(f[0][j & 1], f[1][j >> 1].re, f[1][j >> 1].im);
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const C2<T> d = mulc(e, f[2][b].re, f[2][b].im);
            v[j + 4 * b] = mulc(v[j + 4 * b], d.re, d.im);
          }
        }
      };
      using I0 = std::integral_constant<int, 0>;
      using I1 = std::integral_constant<int, 1>;
      using I2 = std::integral_constant<int, 2>;
      using I3 = std::integral_constant<int, 3>;
      using I4 = std::integral_constant<int, 4>;
      static_assert(kFlipOwnX[0] == 0 && kFlipOwnX[1] == 1 && kFlipOwnX[2] == 3 && kFlipOwnX[3] == 2, "X owners");
      static_assert(kFlipOwnZ[0] == 1 && kFlipOwnZ[1] == 3 && kFlipOwnZ[2] == 2 && kFlipOwnZ[3] == 0, "Z owners");
      chain(I0{}, I0{}, I1{}, I3{}, I2{});
      small_wht_all(v, lane);
      chain(I4{}, I1{}, I3{}, I2{}, I0{});
      if (r + 1 < R) small_wht_all(v, lane);
      __syncthreads();  // S.u and the noisy tables are written again
    }
    if (TRACE && regs_out) {
      // amplitude x of the logical frame sits at x ^ phz, with the sign of neg
      // and of phx there
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        uint32_t g = gl;
#pragma unroll
        for (int k = 0; k < 3; ++k)
          if ((j >> k) & 1) g |= 1u << kFlipRegQubit[k];
        const bool minus = ((__popc(g & phx) ^ neg) & 1) != 0;
        regs_out[((size_t)t << kN) + (g ^ phz)] = minus ? C2<T>{-v[j].re, -v[j].im} : v[j];
      }
    }
    // final Z measurement, highest label first: the norms summed over the
    // lower qubits level by level (register bits 0, 1, 2: qubits 0, 2, 8),
    // each level's conditional probability compared with its draw by a vote
    // in every branch, the votes walked from qubit 8 down
    {
      const double uf = lane < kN ? uniform(seed, tg, (uint64_t)R * (uint64_t)draws_round + (uint64_t)lane) : 0.0;
      auto draw = [&](int q) { return lane_value(uf, kN - 1 - q); };  // level of qubit q
      auto flip = [&](int q) { return (phz >> q) & 1; };
      auto vote = [&](int q, double num, double den) { return __ballot(draw(q) < clamp_p1(num / den)); };
      double n0[8], n1[4], n2[4], n3[2];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const double re = (double)v[j].re, im = (double)v[j].im;
        n0[j] = fma(re, re, im * im);
      }
      // qubit 0 (register bit 0): votes by (qubit 2, qubit 8)
      uint64_t b0[4], b1[4], b2[2], b3[2], b4[2], b5[2], b6[2], b7[2], b8;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        n1[j] = n0[2 * j] + n0[2 * j + 1];
        b0[j] = vote(0, flip(0) ? n0[2 * j] : n0[2 * j + 1], n1[j]);
      }
      // the logical outcome 1 of a lane qubit is its physical bit 1 ^ flip: a
      // lane votes for its own bit, the walk reads the lane with that bit
#pragma unroll
      for (int j = 0; j < 4; ++j) {  // qubit 1 (lane bit 0)
        n2[j] = n1[j] + small_xor<0>(n1[j]);
        b1[j] = vote(1, n1[j], n2[j]);
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {  // qubit 2 (register bit 1): j is qubit 8
        n3[j] = n2[2 * j] + n2[2 * j + 1];
        b2[j] = vote(2, flip(2) ? n2[2 * j] : n2[2 * j + 1], n3[j]);
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {  // qubits 3 .. 7 (lane bits 1 .. 5)
        const double a = n3[j] + small_xor<1>(n3[j]);
        b3[j] = vote(3, n3[j], a);
        const double b = a + small_xor<2>(a);
        b4[j] = vote(4, a, b);
        const double c = b + small_xor<3>(b);
        b5[j] = vote(5, b, c);
        const double d = pair_sum<false>(c);
        b6[j] = vote(6, c, d);
        const double e = pair_sum<true>(d);
        b7[j] = vote(7, d, e);
        n3[j] = e;
      }
      b8 = vote(8, flip(8) ? n3[0] : n3[1], n3[0] + n3[1]);
      uint32_t out = 0;  // logical outcomes
      int l = 0;         // physical lane bits chosen so far
      const int o8 = (int)(b8 & 1), r8 = o8 ^ (int)flip(8);
      out |= (uint32_t)o8 << 8;
      auto walk = [&](uint64_t votes, int q, int lb) {
        const int o = (int)((votes >> (l | (((int)flip(q) ^ 1) << lb))) & 1);
        out |= (uint32_t)o << q;
        l |= (o ^ (int)flip(q)) << lb;
      };
      walk(r8 ? b7[1] : b7[0], 7, 5);
      walk(r8 ? b6[1] : b6[0], 6, 4);
      walk(r8 ? b5[1] : b5[0], 5, 3);
      walk(r8 ? b4[1] : b4[0], 4, 2);
      walk(r8 ? b3[1] : b3[0], 3, 1);
      const int o2 = (int)(((r8 ? b2[1] : b2[0]) >> l) & 1), r2 = o2 ^ (int)flip(2);
      out |= (uint32_t)o2 << 2;
      const uint64_t q1 = r8 ? (r2 ? b1[3] : b1[2]) : (r2 ? b1[1] : b1[0]);
      walk(q1, 1, 0);
      const uint64_t q0 = r8 ? (r2 ? b0[3] : b0[2]) : (r2 ? b0[1] : b0[0]);
      out |= (uint32_t)((q0 >> l) & 1);
      if (lane < kN) bits[(size_t)t * kN + lane] = (uint8_t)((out >> lane) & 1);
    }
    __syncthreads();  // the tables are rewritten by the next trajectory
  }
}

}  // namespace qec
