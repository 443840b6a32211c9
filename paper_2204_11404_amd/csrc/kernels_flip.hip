// Register passes with a basis change (runs without the data ZZ layer).
//
// Without that layer nothing but the checks acts between measurements, and a
// check's Kraus operator is diagonal (up to an XOR permutation) in its own
// basis: the Hadamard basis of its qubits for an X check, the computational
// one for a Z check.  So the register is kept in a mixed basis, some qubits
// transformed and some not, and a chain of consecutive checks whose qubits
// all sit in the right basis is pointwise on the amplitude index whatever
// its types: the norms of every outcome string come out of one read, as for a
// chain of Z checks.  One pass (k_flip):
//   1. applies the decided chain A (a diagonal) and 1/sqrt(S_m),
//   2. transforms up to 12 qubits (the "flips": Walsh-Hadamard, normalised),
//   3. writes the register in place and sums the chain B, whose qubits the
//      flips have brought into its basis.
// No outcome is predicted and nothing is redone.  Every qubit has to change
// basis twice a round; a tile of 2^12 amplitudes keeps the three lowest bits
// for its lanes (runs of 8 amplitudes) and flips nine others, so a round of
// d = 5 (44 flips beside the three lowest bits) takes five passes and one of
// d = 4 three.  (A tile of 2^13 or shorter runs would still need five, one of
// 2^14 four, with one workgroup a compute unit.)
//
// Bound: HBM, one read and one write of the register a pass.  d = 5, p =
// 2e-3: complex128 198-210 us a pass (5.1-5.4 TB/s; the pass without flips
// 193 us, an in-place scale of 512 MiB 192 us), complex64 102-109 us
// (4.9-5.3 TB/s; 95 us without flips).  Above that rate lie the waits between
// a tile's load, regroup and store.  A round: complex64 1.55 -> 0.53 ms,
// complex128 2.4 -> 1.04 ms against the eight speculative passes and their
// redos; 4096 d = 4 trajectories (complex64) 42.7 -> 18.5 ms.
//
// Pauli frames: the XOR permutations are not carried out.  The stored
// register is s Z^phix X^phiz |psi> written in the mixed basis; a Z member
// moves F into phiz, an X member moves F into phix and turns the sign s by
// the parity of F & phiz.
#pragma once

#include "kernels.hip"

namespace qec {

// Walsh-Hadamard stage over lane bit B (0..2): one exchange and one fused
// multiply-add per component (lanes with the bit set keep partner - own).
template <int B>
__device__ __forceinline__ uint32_t lane_xor_u32(uint32_t x) {
  if constexpr (B == 0) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, false);  // quad_perm 1,0,3,2
  } else if constexpr (B == 1) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, false);  // quad_perm 2,3,0,1
  } else {
    // lane ^ 4: banks 0 and 2 (lanes 0-3, 8-11 of a row) read four lanes
    // up, banks 1 and 3 four lanes down
    const int up = __builtin_amdgcn_update_dpp((int)x, (int)x, 0x104, 0xF, 0x5, false);  // row_shl:4
    return (uint32_t)__builtin_amdgcn_update_dpp(up, (int)x, 0x114, 0xF, 0xA, false);    // row_shr:4
  }
}
template <int B, typename T>
__device__ __forceinline__ T lane_xor(T v) {
  constexpr int W = sizeof(T) / 4;
  uint32_t x[W];
  __builtin_memcpy(x, &v, sizeof(T));
#pragma unroll
  for (int i = 0; i < W; ++i) x[i] = lane_xor_u32<B>(x[i]);
  __builtin_memcpy(&v, x, sizeof(T));
  return v;
}
template <int B, typename T>
__device__ __forceinline__ void flip_lane(C2<T>* v, int tid) {
  const T sg = ((tid >> B) & 1) ? (T)-1 : (T)1;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const T ore = lane_xor<B>(v[j].re), oim = lane_xor<B>(v[j].im);
    v[j].re = fma(v[j].re, sg, ore);
    v[j].im = fma(v[j].im, sg, oim);
  }
}

// Walsh-Hadamard stages over the register-slot bits of `mask`.
template <typename T>
__device__ __forceinline__ void flip_slots(C2<T>* v, int mask) {
  if (mask & 1) wht_reg_stage<1>(v);
  if (mask & 2) wht_reg_stage<2>(v);
  if (mask & 4) wht_reg_stage<4>(v);
  if (mask & 8) wht_reg_stage<8>(v);
}

template <typename T> struct FlipBuf { using E = T; };
template <> struct FlipBuf<float> { using E = C2<float>; };

// complex128 holds two copies of a tile, the one it works on and the next
// one's loads in flight, and runs two waves per SIMD; complex64 runs three
// and relies on them (d = 5, mean of a round's passes: complex128 236 us
// without the loads ahead, 212 with; complex64 113 us, 116 with).
template <typename T> struct FlipShape {
  static constexpr int kWaves = sizeof(T) == 8 ? 2 : 3;
  static constexpr bool kAhead = sizeof(T) == 8;
};

// kFlipPass: the steps above.  The first two passes of a trajectory know the
// register without reading it: kFlipSums sums B over the initial code state
// (nothing is stored), kFlipFirst applies A to that state as it forms it.
// The last pass (LB = 0) only sums the final measurement's chunks (keep: it
// stores the register): k_final_measure applies A to the chunk it reads.
// d = 5: the two 155 -> 108 us in complex64 and 297 -> 171 in complex128, the
// last one 96 -> 53 and 194 -> 142 (with k_final_measure 117 -> 88 and 217 -> 180).
// Sums: a partial of every sum per workgroup, or per tile (per_tile: at most
// four tiles a workgroup) where the workgroups of a register depend on how many
// run side by side: the decisions then add the same numbers in the same order
// whatever that is.
template <typename T, int LB, int MODE, bool L5>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FlipShape<T>::kWaves))) void k_flip(
    T* __restrict__ st, const FlipPass* __restrict__ pd, const BlockRT* __restrict__ rta,
    const BlockRT* __restrict__ rtb, const Decision* __restrict__ dec_a, Decision* __restrict__ dec_b,
    double* __restrict__ partials, int reverse, int n_cls_wg, int per_tile, double* __restrict__ chunk_sums,
    int keep, SlotStrides ss) {
  constexpr bool INIT = MODE == kFlipSums, FIRST = MODE == kFlipFirst;
  constexpr uint32_t kAmp = 2 * sizeof(T);
  constexpr bool kAhead = FlipShape<T>::kAhead && MODE == kFlipPass;
  const size_t slot = reverse ? gridDim.y - 1 - blockIdx.y : blockIdx.y;
  st += slot * ss.st;
  if (rta) rta += slot * ss.rt;
  if (rtb) rtb += slot * ss.rt;
  if (dec_a) dec_a += slot * ss.dec;
  dec_b += slot * ss.dec;
  const int n_outer = pd->n_outer, n_brel = pd->n_brel;
  const uint32_t n_cols = per_tile ? 1u << n_outer : gridDim.x;
  partials += slot * kChainAcc * n_cols;
  if (chunk_sums) chunk_sums += slot << n_outer;
  const RegBuf<T> reg(st, (uint32_t)(kAmp << (kTileMax + n_outer)));
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int la = pd->la;

  using E = typename FlipBuf<T>::E;
  static_assert(sizeof(E) == 8, "places are eight bytes");
  __shared__ __align__(16) E buf[FlipLds::kSize];
  __shared__ cd pt[INIT ? 1 : kChainMax / 2][INIT ? 1 : 256];  // A's decided diagonals, two members a table
  __shared__ double wt[LB > 0 ? LB : 1][2][16];

  // frames: after A (recorded for B's decision), and B's member offsets
  uint32_t phz = 0, phx = 0, ca = 0, cb = 0;
  int neg = 0, mbits = 0;
  double scale = pd->norm;
  const T amp = (T)pd->amp;
  if constexpr (!INIT) {
    phz = dec_a->phi;
    phx = dec_a->phix;
    neg = dec_a->neg;
    mbits = dec_a->m;
    scale = pd->norm / sqrt(dec_a->Sm);
    for (int i = 0; i < la; ++i) {
      const bool x = (pd->ax >> i) & 1;
      ca |= gather_loc(x ? phx : phz, pd->aq[i], pd->aw[i]) << (4 * i);
      const uint32_t G = scatter_loc(rta[i].F, pd->aq[i], pd->aw[i]);
      if (x) {
        neg ^= __popc(G & phz) & 1;
        phx ^= G;
      } else {
        phz ^= G;
      }
    }
  }
  if constexpr (LB > 0) {
    uint32_t bz = phz, bx = phx;
    for (int i = 0; i < LB; ++i) {
      const bool x = (pd->bx >> i) & 1;
      cb |= gather_loc(x ? bx : bz, pd->bq[i], pd->bw[i]) << (4 * i);
      const uint32_t G = scatter_loc(rtb[i].F, pd->bq[i], pd->bw[i]);
      (x ? bx : bz) ^= G;
    }
  }
  if (blockIdx.x == 0 && tid == 0) {
    dec_b->phi = phz;
    dec_b->phix = phx;
    dec_b->neg = neg;
  }
  if constexpr (!INIT) {
    for (int k = 0; 2 * k < la; ++k) {
      auto entry = [&](int i, int x) {
        if (i >= la) return cd{1.0, 0.0};
        // an X check's table holds 2^-w for two unnormalised transforms
        const double f = ((pd->ax >> i) & 1) ? (double)(1 << pd->aw[i]) : 1.0;
        const double* d = rta[i].D[(mbits >> i) & 1][x];
        return cd{d[0] * f, d[1] * f};
      };
      cd v = cmul(entry(2 * k, tid & 15), entry(2 * k + 1, tid >> 4));
      if (k == 0) v = cscale(v, scale);
      pt[k][tid] = v;
    }
  }
  if (LB > 0 && tid < LB * 32) {
    const int i = tid >> 5, m = (tid >> 4) & 1, x = tid & 15;
    wt[i][m][x] = rtb[i].W[m][x] * (((pd->bx >> i) & 1) ? (double)(1 << pd->bw[i]) : 1.0);
  }
  __syncthreads();

  const int m0 = pd->m0, m2 = pd->m2, low = pd->low, two = pd->two, touch = pd->touch;
  uint32_t g1 = (uint32_t)(tid & 7), g2 = g1, pa = ca, pb = cb;
  {
    const uint32_t t1[5] = {pd->s2[0], pd->s2[1], pd->e, pd->s2[2], pd->s2[3]};
    const uint32_t t2[5] = {pd->s0[0], pd->s0[1], pd->s0[2], pd->s0[3], pd->e};
#pragma unroll
    for (int i = 0; i < 5; ++i)
      if ((tid >> (3 + i)) & 1) {
        g1 |= t1[i];
        g2 |= t2[i];
      }
    if (!two) g2 = g1;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if ((tid >> i) & 1) {
        pa ^= pd->a_tid[i];
        pb ^= pd->b_tid[i];
      }
  }
  const int lr = (tid & 7) + ((tid >> 3) & 1) * FlipLds::s0[0] + ((tid >> 4) & 1) * FlipLds::s0[1] +
                 ((tid >> 5) & 1) * FlipLds::s0[2] + ((tid >> 6) & 1) * FlipLds::s0[3] + ((tid >> 7) & 1) * FlipLds::e;
  const int lw = (tid & 7) + ((tid >> 3) & 1) * FlipLds::s2[0] + ((tid >> 4) & 1) * FlipLds::s2[1] +
                 ((tid >> 5) & 1) * (L5 ? FlipLds::s0[3] : FlipLds::e) + ((tid >> 6) & 1) * FlipLds::s2[2] +
                 ((tid >> 7) & 1) * FlipLds::s2[3];
  // byte places: a thread's part XOR a slot's (uniform) XOR a tile's
  auto in_place = [](uint32_t g) { return flip_place<T>(g) * kAmp; };
  auto out_place = [&](uint32_t g) { return (pd->plain ? g : flip_place<T>(g)) * kAmp; };
  uint32_t o1[4], o2[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    o1[b] = in_place(pd->s0[b]);
    o2[b] = out_place(two ? pd->s2[b] : pd->s0[b]);
  }
  const uint32_t p1 = in_place(g1), p2 = out_place(g2);
  auto at = [](const uint32_t* o, int j) {
    return (j & 1 ? o[0] : 0u) ^ (j & 2 ? o[1] : 0u) ^ (j & 4 ? o[2] : 0u) ^ (j & 8 ? o[3] : 0u);
  };

  // The workgroup's tiles: classes agree in the outer bits that carry qubits
  // of B (n_cls_wg workgroup groups share them out), steps run through the
  // other outer bits.  Within a class the norms of the 16 slots add up; B's
  // weights enter once a class.
  const uint32_t n_cls = 1u << n_brel, n_steps = 1u << (n_outer - n_brel);
  const uint32_t c0 = blockIdx.x % n_cls_wg, w0 = blockIdx.x / n_cls_wg, gs = gridDim.x / n_cls_wg;
  // (global bits of a tile, and A's packed index there)
  auto tile_of = [&](uint32_t c, uint32_t step) { return ((reverse ? n_steps - 1 - step : step) << n_brel) | c; };
  auto locate = [&](uint32_t c, uint32_t step, uint32_t& b, uint32_t& x) {
    const uint32_t tile = tile_of(c, step);
    b = x = 0;
    for (int i = 0; i < n_outer; ++i)
      if ((tile >> i) & 1) {
        b |= pd->outer_bit[i];
        x ^= pd->a_outer[i];
      }
  };
  double acc[LB > 0 ? 16 : 1];
#pragma unroll
  for (int j = 0; j < (LB > 0 ? 16 : 1); ++j) acc[j] = 0.0;
  constexpr int kN = LB > 0 ? 1 << LB : 1, kGroups = kN > 16 ? kN / 16 : 1;
  // lane l: sum (l >> 2) & 15 of each group of 16 (per_tile: of tile l & 3)
  double total[kGroups];
  int n_sums = 0;  // per_tile: tiles summed
#pragma unroll
  for (int k = 0; k < kGroups; ++k) total[k] = 0.0;

  // the initial state's linear conditions: parts of the thread and the slots;
  // its sign, a quadratic form of the index, over the 16 slots as a bit mask:
  // the slots' own part here, what a tile and a thread add to it is linear in
  // the slot
  uint32_t syn_t = 0, rep_t = 0, syn_s[4] = {}, rep_s[4] = {}, sign_s = 0;
  int count[INIT ? 16 : 1];
#pragma unroll
  for (int j = 0; j < (INIT ? 16 : 1); ++j) count[j] = 0;
  auto lin = [&](uint32_t g, uint32_t& syn, uint32_t& rep) {
    uint32_t c = 0;
    for (int i = 0; i < pd->n_piv; ++i)
      if (g & pd->piv_bit[i]) c ^= pd->piv_vec[i];
    syn = (c ^ g) & pd->zmask;
    rep = c & ~pd->zmask;
    for (int i = 0; i < pd->n_par; ++i) syn ^= (uint32_t)(__popc(g & pd->par_vec[i]) & 1) << pd->par_pos[i];
  };
  if constexpr (INIT || FIRST) {
    lin(g1, syn_t, rep_t);
#pragma unroll
    for (int b = 0; b < 4; ++b) lin(pd->s0[b], syn_s[b], rep_s[b]);
    for (int j = 0; j < 16; ++j) sign_s |= (uint32_t)(__popc(at(pd->s0, j) & at(rep_s, j)) & 1) << j;
  }

  C2<T> nv[kAhead ? 16 : 1];
  uint32_t cls = c0, step = w0, base = 0, xa = 0, nbase = 0, nxa = 0;
  locate(cls, step, nbase, nxa);
  auto fetch = [&](C2<T>* d, uint32_t b) {
    const uint32_t w = in_place(b) ^ p1;
#pragma unroll
    for (int j = 0; j < 16; ++j) d[j] = reg.ld(w ^ at(o1, j), 0);
  };
  if constexpr (kAhead) fetch(nv, nbase);
  for (bool more = true; more;) {
    base = nbase;
    xa = nxa;
    C2<T> v[16];
    if constexpr (kAhead) {
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = nv[j];
    }
    const uint32_t cls_now = cls;
    step += gs;
    if (step >= n_steps) {
      step = w0;
      cls += n_cls_wg;
      more = cls < n_cls;
    }
    if (more) {
      locate(cls, step, nbase, nxa);
      if constexpr (kAhead) fetch(nv, nbase);
    }
    uint32_t on = 0;
    if constexpr (INIT || FIRST) {
      // the initial code state in the mixed basis it starts in: amplitude g is
      // +-amp where every linear condition holds; its sign is the parity of
      // the transformed bits and of the code word that matches the
      // untransformed ones
      uint32_t syn_b, rep_b;
      lin(base, syn_b, rep_b);
      syn_b ^= syn_t;
      rep_b ^= rep_t;
      if constexpr (INIT) {
#pragma unroll
        for (int j = 0; j < 16; ++j) count[j] += syn_b == at(syn_s, j) ? 1 : 0;
      } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) on |= syn_b == at(syn_s, j) ? 1u << j : 0u;
        const uint32_t gb = base | g1;
        const uint32_t lines[4] = {0xAAAAu, 0xCCCCu, 0xF0F0u, 0xFF00u};
        uint32_t minus = sign_s ^ ((__popc(gb & rep_b) & 1) ? 0xFFFFu : 0u);
#pragma unroll
        for (int b = 0; b < 4; ++b)
          if ((__popc(gb & rep_s[b]) ^ __popc(pd->s0[b] & rep_b)) & 1) minus ^= lines[b];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const T a = (on >> j) & 1 ? amp : (T)0;
          v[j] = C2<T>{(minus >> j) & 1 ? -a : a, (T)0};
        }
      }
    } else if constexpr (!kAhead) {
      fetch(v, base);
    }
    // (FIRST: a wave without an amplitude stays zero until the regroup)
    const bool some = !FIRST || __ballot(on != 0) != 0;
    if constexpr (!INIT) {
      if (some) {
        // chain A: the tables that see the same index in all 16 slots as one
        // factor, the others slot by slot
        const uint32_t oa = pa ^ xa;
        cd f{1.0, 0.0};
#pragma unroll
        for (int k = 0; k < kChainMax / 2; ++k)
          if (2 * k < la && !((touch >> k) & 1)) f = cmul(f, pt[k][(oa >> (8 * k)) & 255]);
        if (touch == 0) {
          const T fr = (T)f.re, fi = (T)f.im;
#pragma unroll
          for (int j = 0; j < 16; ++j) v[j] = FIRST ? C2<T>{v[j].re * fr, v[j].re * fi} : mulc(v[j], fr, fi);
        } else {
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const uint32_t oj = oa ^ at(pd->a_slot, j);
            cd e = f;
#pragma unroll
            for (int k = 0; k < kChainMax / 2; ++k)
              if ((touch >> k) & 1) e = cmul(e, pt[k][(oj >> (8 * k)) & 255]);
            v[j] = FIRST ? C2<T>{v[j].re * (T)e.re, v[j].re * (T)e.im} : mulc(v[j], (T)e.re, (T)e.im);
          }
        }
        flip_slots(v, m0);
        if (low & 1) flip_lane<0>(v, tid);
        if (low & 2) flip_lane<1>(v, tid);
        if (low & 4) flip_lane<2>(v, tid);
        if constexpr (L5) {
          // e, on lane bit 5, changes places with slot bit 3
#pragma unroll
          for (int j = 0; j < 8; ++j) swap_c2<T, true>(v[j], v[j + 8]);
          wht_reg_stage<8>(v);
        }
      }
      if (two) {
        E* const bw = buf + lw;
        const E* const br = buf + lr;
        if constexpr (sizeof(T) == 4) {
          __syncthreads();
#pragma unroll
          for (int j = 0; j < 16; ++j) bw[FlipLds::w<L5>(j)] = v[j];
          __syncthreads();
#pragma unroll
          for (int j = 0; j < 16; ++j) v[j] = br[FlipLds::r(j)];
        } else {
          __syncthreads();
#pragma unroll
          for (int j = 0; j < 16; ++j) bw[FlipLds::w<L5>(j)] = v[j].re;
          __syncthreads();
#pragma unroll
          for (int j = 0; j < 16; ++j) v[j].re = br[FlipLds::r(j)];
          __syncthreads();
#pragma unroll
          for (int j = 0; j < 16; ++j) bw[FlipLds::w<L5>(j)] = v[j].im;
          __syncthreads();
#pragma unroll
          for (int j = 0; j < 16; ++j) v[j].im = br[FlipLds::r(j)];
        }
        flip_slots(v, m2);
      }
      if (LB > 0 || keep) {
        const uint32_t w = out_place(base) ^ p2;
#pragma unroll
        for (int j = 0; j < 16; ++j) reg.st(w ^ at(o2, j), 0, v[j]);
      }
    }
    if constexpr (LB > 0) {
      if constexpr (!INIT) {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const double re = (double)v[j].re, im = (double)v[j].im;
          acc[j] = fma(re, re, fma(im, im, acc[j]));
        }
      }
      if (!more || cls != cls_now || per_tile) {
        if constexpr (INIT) {
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            acc[j] = (double)count[j] * ((double)amp * (double)amp);
            count[j] = 0;
          }
        }
        // the class's norms against B's weights: the two members that slot
        // bits belong to take those bits in (16 norms -> four, one per pair
        // of their outcomes), the other members' weights are the thread's own
        uint32_t ob = pb;
        for (int i = 0; i < n_brel; ++i)
          if ((cls_now >> i) & 1) ob ^= pd->b_outer[i];
        double z[4];
        {
          const int mp = pd->ord[LB >= 2 ? LB - 2 : 0], mq = pd->ord[LB - 1];
          const uint32_t xp = (ob >> (4 * mp)) & 15u, xq = (ob >> (4 * mq)) & 15u;
          double y[2][4];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            double u[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) u[c] = wt[mp][h][xp ^ ((at(pd->b_slot, c) >> (4 * mp)) & 15u)];
#pragma unroll
            for (int q = 0; q < 4; ++q)
              y[h][q] = u[0] * acc[4 * q] + u[1] * acc[4 * q + 1] + u[2] * acc[4 * q + 2] + u[3] * acc[4 * q + 3];
          }
          if constexpr (LB >= 2) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              double u[4];
#pragma unroll
              for (int c = 0; c < 4; ++c) u[c] = wt[mq][h][xq ^ ((at(pd->b_slot, 4 * c) >> (4 * mq)) & 15u)];
#pragma unroll
              for (int k = 0; k < 2; ++k)
                z[k + 2 * h] = u[0] * y[k][0] + u[1] * y[k][1] + u[2] * y[k][2] + u[3] * y[k][3];
            }
          } else {  // a single check: its other slot bits carry nothing
#pragma unroll
            for (int k = 0; k < 2; ++k) z[k] = (y[k][0] + y[k][1]) + (y[k][2] + y[k][3]);
            z[2] = z[3] = 0.0;
          }
        }
        constexpr int R = LB >= 2 ? LB - 2 : 0;  // members without slot bits
        double p[1 << R];
        p[0] = 1.0;
#pragma unroll
        for (int l = 0; l < R; ++l) {
          const int m = pd->ord[l];
          const uint32_t x = (ob >> (4 * m)) & 15u;
          const double u0 = wt[m][0][x], u1 = wt[m][1][x];
#pragma unroll
          for (int h = 0; h < (1 << l); ++h) {
            p[h + (1 << l)] = p[h] * u1;
            p[h] *= u0;
          }
        }
        // sum number r + 2^R (outcome of mp + 2 outcome of mq)
#pragma unroll
        for (int k = 0; k < kGroups; ++k) {
          double t[16];
#pragma unroll
          for (int a = 0; a < 16; ++a) {
            const int n = 16 * k + a;
            t[a] = n < kN ? p[n & ((1 << R) - 1)] * z[(n >> R) & 3] : 0.0;
          }
          const double w = wave_reduce16(t);
          if (!per_tile) total[k] += w;
          else if ((lane & 3) == n_sums) total[k] = w;
        }
        ++n_sums;
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[j] = 0.0;
      }
    } else if (chunk_sums) {
      // the last pass of a trajectory: its tiles are the chunks of the final
      // measurement
      double s = 0.0;
#pragma unroll
      for (int j = 0; j < 16; ++j) s += (double)v[j].re * (double)v[j].re + (double)v[j].im * (double)v[j].im;
      s = wave_sum(s);
      __syncthreads();
      if (lane == 0) wt[0][0][wid] = s;
      __syncthreads();
      if (tid == 0) chunk_sums[base >> kTileMax] = (wt[0][0][0] + wt[0][0][1]) + (wt[0][0][2] + wt[0][0][3]);
    }
  }

  if constexpr (LB > 0) {
    // the waves' totals added up, a column of the partial sums per workgroup
    // or tile
    double(*const red)[kN][4] = reinterpret_cast<double(*)[kN][4]>(buf);
    const int n_own = per_tile ? n_sums : 1;
    __syncthreads();  // the regroup buffer is read no more
#pragma unroll
    for (int k = 0; k < kGroups; ++k)
      if ((lane & 3) < n_own && 16 * k + (lane >> 2) < kN) red[lane & 3][16 * k + (lane >> 2)][wid] = total[k];
    __syncthreads();
    const int own = tid >> LB, n = tid & (kN - 1);  // (at most 4 x 64 of the 256 threads)
    const uint32_t own_steps = (n_steps - w0 + gs - 1) / gs;
    const uint32_t col = per_tile ? tile_of(c0 + own / own_steps * n_cls_wg, w0 + own % own_steps * gs) : blockIdx.x;
    if (own < n_own) {
      uint32_t h = 0;  // outcome bits in member order
#pragma unroll
      for (int l = 0; l < LB; ++l) h |= ((n >> l) & 1) << pd->ord[l];
      const double s = (red[own][n][0] + red[own][n][1]) + (red[own][n][2] + red[own][n][3]);
      // sums of a chain of one or two are laid out as every prefix's
      partials[(size_t)(LB == 2 ? 2 + h : h) * n_cols + col] = s;
    }
    if constexpr (LB == 2) {
      if (own < n_own && n < 2) {  // outcome n of member 0, either outcome of member 1
        double s = 0.0;
        const int o = pd->ord[0] == 0 ? 1 : 2;
        for (int w = 0; w < 4; ++w) s += red[own][n * o][w] + red[own][n * o + 3 - o][w];
        partials[(size_t)n * n_cols + col] = s;
      }
    }
  }
}

}  // namespace qec
