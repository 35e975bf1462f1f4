// qd_rollout.hpp -- policy rollouts on the synthetic dynamics (gfx950).
//
// Evaluation of a batch of tanh MLP policies (two hidden tanh layers and a
// tanh output, as in Section 5.1 of the paper) for T steps of
// s' = tanh(A s + B a).  Every individual has its own weights, so this is a
// batch of independent GEMV chains, not one GEMM: no matrix core applies.
//
// One, two or eight waves run one individual with all its weights in VGPRs for
// the whole episode.  The summation order of every output is fixed (hidden
// layers and A s: four interleaved partial sums, then the bias; output layer: 8
// slices folded pairwise, then the bias; dynamics: A s + B a), which keeps the
// result independent of the launch shape.
//
// The genotype is produced in the kernel's prologue straight from the parents
// (or the Glorot-uniform first batch) -- offspring weights never touch HBM.
#pragma once

#include "qd_kernels.hpp"

namespace qd {

constexpr int kObs = 27, kAct = 8;

inline bool rollout_supported(int obs, int hid, int act) {
  return obs == kObs && act == kAct && (hid == 64 || hid == 128);
}

// Glorot-uniform first-batch gene i (biases are zero).
__device__ __forceinline__ float mlp_init_gene(const Params& p, int i, float u) {
  const int o = p.obs, h = p.hid, a = p.act;
  const int e1 = h * o, e2 = e1 + h, e3 = e2 + h * h, e4 = e3 + h, e5 = e4 + a * h;
  float lim;
  if (i < e1) lim = __builtin_sqrtf(6.0f / (float)(o + h));
  else if (i < e2) lim = 0.0f;
  else if (i < e3) lim = __builtin_sqrtf(6.0f / (float)(h + h));
  else if (i < e4) lim = 0.0f;
  else if (i < e5) lim = __builtin_sqrtf(6.0f / (float)(h + a));
  else lim = 0.0f;
  return lim == 0.0f ? 0.0f : fma32(u, lim + lim, -lim);
}

// Genes 4 blk .. 4 blk + 3 of policy offspring j.
template <bool GEN0>
__device__ __forceinline__ float4 mlp_gene_block(const Params& p, const Pair& q, uint32_t g, int j,
                                                 int blk) {
  if (GEN0) {
    const uint4 x = philox((uint32_t)blk, (uint32_t)j, 0u, kTagInit, p.key);
    const int i = 4 * blk;
    return make_float4(mlp_init_gene(p, i, unit24(x.x)), mlp_init_gene(p, i + 1, unit24(x.y)),
                       mlp_init_gene(p, i + 2, unit24(x.z)), mlp_init_gene(p, i + 3, unit24(x.w)));
  }
  return make_genes<false>(p, q, g, j, 4 * blk);
}

// The layers' dot products: four interleaved partial sums (input k goes to
// partial k mod 4, each an fma chain in input order from 0), folded as
// (p0 + p2) + (p1 + p3).
//
// A quad of lanes shares R rows (neurons) of a layer and lane t of the quad
// runs partial t of every one of them, so a lane needs the inputs 4 m + t
// only: N / 4 of the N inputs, read once and used for R rows.  With the inputs
// in LDS as [t][m], a float4 read serves 4 R fmas -- plain v_fmac on vector
// registers, which the SIMD issues two at a time, where a broadcast inside the
// instruction (DPP) or a scalar operand is issued one at a time.
// Accumulator r of lane t belongs to row r ^ (t mod R) of the quad: with that
// order the fold needs no select, and (for R = 4) lane t ends with row t.
template <int CTRL>
__device__ __forceinline__ float quad_perm(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float quad_xor1(float v) { return quad_perm<0xb1>(v); }   // [1,0,3,2]
__device__ __forceinline__ float quad_xor2(float v) { return quad_perm<0x4e>(v); }   // [2,3,0,1]

// Sum of the row that lane t of a quad ends with: row t (R = 4), row t mod 2
// (R = 2), the quad's row (R = 1).  Each addition is one of (p0 + p2) + (p1 + p3)
// up to the order of its two operands.
template <int R>
__device__ __forceinline__ float quad_fold(const float (&acc)[R]) {
  static_assert(R == 1 || R == 2 || R == 4, "rows per quad");
  if constexpr (R == 4) {
    const float b0 = acc[0] + quad_xor2(acc[2]), b1 = acc[1] + quad_xor2(acc[3]);
    return b0 + quad_xor1(b1);
  } else if constexpr (R == 2) {
    const float b0 = acc[0] + quad_xor2(acc[0]), b1 = acc[1] + quad_xor2(acc[1]);
    return b0 + quad_xor1(b1);
  } else {
    const float b0 = acc[0] + quad_xor2(acc[0]);
    return b0 + quad_xor1(b0);
  }
}

// The T at byte offset `at` (a lane's own, in one register) from p (the same in
// every lane, folded into the instruction).
template <class T>
__device__ __forceinline__ const T& lds_at(const float* p, int at) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + at);
}

__device__ __forceinline__ float& lds_ref(float* p, int at) {
  return *reinterpret_cast<float*>(reinterpret_cast<char*>(p) + at);
}

// M inputs of this lane's partial for R rows, weights w[r][m]; x: the lane's
// [t] row, 16-byte aligned.  LIM inputs' reads are in flight at most.
template <int R, int M, int LIM>
__device__ __forceinline__ float quad_dot(const float (&w)[R][M], const float* x, int at) {
  float acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int m4 = 0; m4 < M; m4 += 4) {
    const float4 v = lds_at<float4>(x + m4, at);
    const float xv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (m4 + i < M) {
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = fma32(w[r][m4 + i], xv[i], acc[r]);
      }
    }
    if (m4 % LIM == LIM - 4 && m4 + 4 < M) {
#pragma unroll
      for (int r = 0; r < R; ++r) __asm__ volatile("" : "+v"(at), "+v"(acc[r]));
    }
  }
  return quad_fold<R>(acc);
}

// The same with the inputs already in registers.
template <int R, int M>
__device__ __forceinline__ float quad_dot(const float (&w)[R][M], const float4 (&x)[(M + 3) / 4]) {
  float acc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) acc[r] = 0.0f;
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const float4& v = x[m / 4];
    const float xm = m % 4 == 0 ? v.x : (m % 4 == 1 ? v.y : (m % 4 == 2 ? v.z : v.w));
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = fma32(w[r][m], xm, acc[r]);
  }
  return quad_fold<R>(acc);
}

// A pair that is the same in every lane of the wave, moved to scalar registers.
__device__ __forceinline__ Pair uniform_pair(const Params& p, const Pair& v) {
  Pair q = v;
  q.c1 = __builtin_amdgcn_readfirstlane(v.c1);
  q.c2 = __builtin_amdgcn_readfirstlane(v.c2);
  q.banks = (uint32_t)__builtin_amdgcn_readfirstlane((int)v.banks);
  q.lambda = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v.lambda)));
  q.row1 = geno_row(p, q.banks & 1u, q.c1);
  q.row2 = geno_row(p, (q.banks >> 1) & 1u, q.c2);
  return q;
}

// Orders the LDS accesses of one individual's NT threads around this point.
template <int NT>
__device__ __forceinline__ void group_sync() {
  if constexpr (NT > 64) __syncthreads();
  else wave_sync();
}

// Steps a rollout records for its reward and descriptor sums (see k_rollout).
constexpr int kRing = 64;

// Folds the first m ring slots into the running sums; called by all 64
// lanes of the output wave (o: lane index in it).  Lane i < m turns slot i
// into its step's reward s'_0 - 0.5 |a|^2 (|a|^2 as an fma chain over the
// actions in order) and the sigmoids of s'_1 .. s'_4; then lane 0 adds the m
// rewards and lanes 1 .. 4 their m sigmoids to `acc`, in slot (= step) order
// -- the same operations in the same order as adding each step's terms as
// the step ends.
template <int A>
__device__ __forceinline__ void flush_ring(float (*ra)[A], float (*rs)[kRing + 1], int m, int o,
                                           float& acc) {
  wave_sync();
  if (o < m) {
    float qa = 0.0f;
#pragma unroll
    for (int k = 0; k < A; ++k) qa = fma32(ra[o][k], ra[o][k], qa);
    rs[0][o] = fma32(-0.5f, qa, rs[0][o]);
#pragma unroll 1
    for (int c = 1; c <= 4; ++c) rs[c][o] = sigmoid32(rs[c][o]);
  }
  wave_sync();
  if (o <= 4) {
    const float* row = rs[o];
    int i = 0;
#pragma unroll 1
    for (; i + 8 <= m; i += 8) {   // eight loads in flight, then eight adds
      float v[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = row[i + t];
#pragma unroll
      for (int t = 0; t < 8; ++t) acc = acc + v[t];
    }
#pragma unroll 1
    for (; i < m; ++i) acc = acc + row[i];
  }
  wave_sync();
}

// One individual per W waves.  Quad u = 16 wave + lane / 4 of its waves holds
// rows R u .. R u + R - 1 of W1 and W2, R = H / (16 W), each lane its partial's
// weights (inputs t, t + 4, ...) of those rows in VGPRs for the whole episode.
// In the last stage of a step lane l holds W3[l mod 8][slice l / 8 of H / 8
// inputs], whose 8 partial sums are folded across the wave, and works on state
// component 2 (l / 4) + (l mod 2) of the new state with that row of B and two
// rows of A (a quad's two state components).
// Per step: layer 1, barrier, layer 2 (and A s, on the other wave than the
// output one), barrier, then on the output wave the output layer, B a and the
// new state, barrier.  With one wave there is no barrier, and with one row per
// quad (R = 1: few individuals, every SIMD has waves to spare) each wave runs
// the last stage for itself, which saves the third one.  The reward and the
// descriptor's sigmoids, which only five lanes need, are not evaluated in the
// step: its actions and new-state components 0 .. 4 go to a ring in LDS, folded
// in every kRing steps by the output wave.
//
// What bounds a step is the length of its chain: a lone wave issues one
// instruction per ~5.3 cycles, and every exchange through LDS adds its latency
// (the state is read into registers as soon as it is written, and A s fills the
// wait for the first layer).  At three waves per SIMD (64 wide) the SIMD issues
// one VALU instruction per ~3 cycles, 280 a step.  Measured, one generation
// with the earlier layout (inputs broadcast inside DPP fmas, a row per lane)
// and this one: 64 wide, T = 250: 256 individuals 230 -> 202 us, 8192: 866 ->
// 763 us (34 -> 39 TFLOP/s); 128 wide, T = 400: 256: 448 -> 391 us, 1501:
// 1052 -> 928 us, 16384: 8165 -> 7420 us.
template <int H, int W>
struct RolloutShape {
  static constexpr int O = kObs, A = kAct, NT = W * 64, R = H / (16 * W);
  // individuals per workgroup: two one-wave individuals share the sampler's
  // table, so that the LDS of a CU holds the 12 that its registers hold
  static constexpr int kInd = W == 1 ? 2 : 1, kThreads = NT * kInd;
  static constexpr int kWavesPerSimd = W == 1 ? 3 : (W == 2 ? 2 : 4);
  static constexpr bool kOwnState = R == 1 && W > 1;     // every wave runs the last stage
  static constexpr bool kShared = W > 1 && !kOwnState;   // the output wave runs it for all
  static constexpr int kSlab = W == 1 ? 8 : 16;          // inputs of W2 per pass of the prologue
  static constexpr int kSlabPitch = kSlab + 4;
  // A vector of N inputs lies in LDS as [t][m], input 4 m + t, rows kPitch
  // apart (padded: the four rows' float4 reads fall in different banks).
  static constexpr int kPitch = H / 4 + 4;
  // The workgroup's LDS in floats: the sampler's table, then per individual the
  // prologue's stage, later the episode's buffers.
  static constexpr int kTab = kNormalRows * 4;
  static constexpr int kRa = 0, kRs = kRa + kRing * A, kX = kRs + (5 * (kRing + 1) + 3) / 4 * 4;
  static constexpr int kXs = kPitch * 4, kH1 = kX + kXs * (kOwnState ? W : 1), kH2 = kH1 + kXs;
  static constexpr int kAs = kH2 + kXs, kFail = kAs + (kShared ? 32 : 0);
  static constexpr int kEpisode = kFail + (kShared ? 4 : 0);
  static constexpr int kW1Stage = H * O, kW2Stage = H * kSlabPitch, kTail = 9 * H + A;
  // Registers beside W1 and W2: the output wave's slice of W3 and row of B, and
  // A's rows on the wave that works out A s -- the same registers where these
  // are different waves.
  static constexpr int kAuxB = 0, kAuxB3 = A, kAuxW3 = A + 1;
  static constexpr int kLast = kAuxW3 + H / 8, kAuxA = kShared ? 0 : kLast;
  static constexpr int max2(int a, int b) { return a > b ? a : b; }
  static constexpr int kAux = max2(kAuxA + 14, kLast);
  static constexpr int kRegion = max2(max2(kEpisode, kW1Stage), max2(kW2Stage, kTail + H));
  static constexpr int kMem = kTab + kInd * kRegion;
};

template <int H, int W, bool GEN0, bool KEEP>
__device__ __forceinline__ void rollout(const Params& p, uint32_t g) {
  using S = RolloutShape<H, W>;
  constexpr int O = S::O, A = S::A, R = S::R, NT = S::NT, SL = H / 8, M1 = (O + 3) / 4, M2 = H / 4;
  constexpr int P = S::kPitch;
  constexpr int E1 = H * O, E2 = E1 + H, E3 = E2 + H * H;   // b1, W2, b2 (then W3, b3)
  static_assert(O == 27 && A == 8, "lane order of the state and the actions");
  __shared__ __attribute__((aligned(16))) float s_mem[S::kMem];
  float4* s_tab = reinterpret_cast<float4*>(s_mem);

  const int tid = threadIdx.x & (NT - 1), lane = threadIdx.x & 63;
  const int ind = S::kInd == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
  const int wave = W == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid >> 6);
  const int t = lane & 3, quad = wave * 16 + (lane >> 2);
  const int row0 = quad * R, flip = t & (R - 1);
  // the last workgroup's spare wave repeats the last individual and stores nothing
  const int jj = (int)blockIdx.x * S::kInd + ind;
  const bool mine = jj < p.nb;
  const int j = mine ? jj : p.nb - 1;
  float* st = s_mem + S::kTab + ind * S::kRegion;
  // Row rho of the R u + r counts neuron 4 (rho mod H/4) + rho / (H/4): the
  // order of the [t][m] layout, so a lane's place in it follows from its lane.
  const auto neuron = [](int rho) { return 4 * (rho & (M2 - 1)) + rho / M2; };
  // The output wave keeps the ring.  Where it runs the last stage for both
  // waves, the other one works out A s for it, and which of the two it is
  // alternates with every 256 workgroups (about one per CU), so that the SIMDs
  // of a CU share that work.
  const int out_wave = S::kShared ? (int)((blockIdx.x >> 8) & 1u) : W - 1;
  const bool is_out = wave == out_wave;
  const bool is_last = !S::kShared || is_out, is_as = !S::kShared || !is_out;

  Pair q{nullptr, nullptr, 0.0f, -1, -1, 0u};
  if (!GEN0) {
    const int nocc = p.counters[0];
    if (nocc <= 0) {
      if (tid == 0 && mine) record_empty_archive(p, j);
      return;
    }
    stage_normal_table(s_tab, p.ntab, (int)threadIdx.x, NT * S::kInd);
    __syncthreads();
    q = uniform_pair(p, select_pair(p, g, j, nocc, Tables{s_tab}));
  }

  // ---- prologue: this individual's genotype, through LDS into registers.  Its
  // gene blocks are made by all its threads; W1 comes last, so that the fewest
  // weights are in registers beside the sampler's.
  const auto make = [&](int blk, float* dst) {
    const float4 v = mlp_gene_block<GEN0>(p, q, g, j, blk);
    *reinterpret_cast<float4*>(dst) = v;
    if (KEEP && mine) *reinterpret_cast<float4*>(p.off_geno + (size_t)j * (size_t)p.stride + 4 * blk) = v;
  };
  float w1[R][M1], w2[R][M2], aux[S::kAux];
  // W2, kSlab inputs of every row a pass
#pragma unroll
  for (int m0 = 0; m0 < M2; m0 += S::kSlab / 4) {
    constexpr int BR = S::kSlab / 4;
#pragma unroll 1
    for (int b = tid; b < H * BR; b += NT) {
      const int row = b / BR, m = b % BR;
      make((E2 + row * H) / 4 + m0 + m, st + row * S::kSlabPitch + 4 * m);
    }
    group_sync<NT>();
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int m = 0; m < BR; ++m) {
        w2[r][m0 + m] = st[neuron(row0 + (r ^ flip)) * S::kSlabPitch + 4 * m + t];
        hold(w2[r][m0 + m]);
      }
    group_sync<NT>();
  }
  // b2, W3, b3, and b1
#pragma unroll 1
  for (int b = tid; b < (S::kTail + H) / 4; b += NT)
    make(b < S::kTail / 4 ? E3 / 4 + b : E1 / 4 + b - S::kTail / 4, st + 4 * b);
  group_sync<NT>();
  const float b1 = st[S::kTail + neuron(row0 + flip)], b2 = st[neuron(row0 + flip)];
  if (is_last) {
#pragma unroll
    for (int i = 0; i < SL; ++i) aux[S::kAuxW3 + i] = st[H + (lane & 7) * H + (lane >> 3) * SL + i];
    aux[S::kAuxB3] = st[9 * H + (lane & 7)];
  }
  group_sync<NT>();
#pragma unroll 1
  for (int b = tid; b < H * O / 4; b += NT) make(b, st + 4 * b);
  group_sync<NT>();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    // input 27 does not exist: -0 times the zero in the state's place 27 adds nothing
#pragma unroll
    for (int m = 0; m < M1; ++m) {
      w1[r][m] = 4 * m + t < O ? st[neuron(row0 + (r ^ flip)) * O + 4 * m + t] : -0.0f;
      hold(w1[r][m]);
    }
  }
  group_sync<NT>();   // every stage is free

  // ---- A, B and the first state
  const int srow = 2 * (lane >> 2) + (lane & 1);   // state component this lane works on
  const bool dyn_lane = srow < O && (lane & 2) == 0;
  const float* envA = p.env;
  const float* envB = p.env + O * O;
  const float* envS = p.env + O * O + O * A;
  // (A's entry 27 of a row is the next row's first, or B's: read and dropped)
  if (is_last) {
    const float* src = envB + (srow < O ? srow : 0) * A;
#pragma unroll
    for (int k = 0; k < A; ++k) aux[S::kAuxB + k] = srow < O ? src[k] : 0.0f;
  }
  if (is_as) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int row = 2 * (lane >> 2) + (r ^ (lane & 1));
      const float* src = envA + (row < O ? row : 0) * O + t;
#pragma unroll
      for (int m = 0; m < M1; ++m) {
        const float v = src[4 * m];
        aux[S::kAuxA + M1 * r + m] = 4 * m + t >= O ? -0.0f : (row < O ? v : 0.0f);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < S::kAux; ++i) hold(aux[i]);
  float (*s_ra)[A] = reinterpret_cast<float (*)[A]>(st + S::kRa);
  float (*s_rs)[kRing + 1] = reinterpret_cast<float (*)[kRing + 1]>(st + S::kRs);
  float* s_x = st + S::kX + (S::kOwnState ? S::kXs * wave : 0);
  float* s_h1 = st + S::kH1;
  float* s_h2 = st + S::kH2;
  float* s_as = st + S::kAs;
  int* s_fail = reinterpret_cast<int*>(st + S::kFail);
  if (lane < 32) {   // places 27 .. 31 of the state stay zero
    const int i = 4 * (lane & 7) + (lane >> 3);
    s_x[(lane >> 3) * P + (lane & 7)] = i < O ? envS[i] : 0.0f;
  }
  if (S::kShared && tid == 0) *s_fail = 0;
  group_sync<NT>();

  // ---- episode; with death_mode != 0 it ends at the first new state whose
  // component 0 is below death_below, and that step counts for nothing.
  // Output-wave lane 0 sums the rewards, lanes 1 .. 4 the sigmoids of state
  // components 1 .. 4, each in step order; both are worked out from the ring,
  // kRing steps at a time (flush_ring), not inside the step.
  // The lane's offsets, kept in one register each: every LDS address in the
  // step is one of them plus a constant.
  int at_part = 4 * t * P;
  int at_row = 4 * ((row0 + flip) + 4 * ((row0 + flip) / M2));
  int at_slice = (lane >> 3) * SL, at_srow = 4 * ((srow & 3) * P + (srow >> 2));
  hold(at_part);
  hold(at_row);
  hold(at_slice);
  hold(at_srow);
  float4 x[2];   // this lane's partial of the state
  const auto read_state = [&]() {
    x[0] = lds_at<float4>(s_x, at_part);
    x[1] = lds_at<float4>(s_x + 4, at_part);
  };
  const auto a_times_s = [&]() {
    float w[2][M1];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
      for (int m = 0; m < M1; ++m) w[r][m] = aux[S::kAuxA + M1 * r + m];
    return quad_dot<2, M1>(w, x);
  };
  float acc = 0.0f;
  int valid = 0;
  bool failed = false;
  read_state();
  for (int step = 0; step < p.T; ++step) {
    const int slot = valid & (kRing - 1);
    const float z1 = quad_dot<R, M1>(w1, x) + b1;
    lds_ref(s_h1, at_row) = tanh32(z1);
    float as = 0.0f;
    if (!S::kShared) as = a_times_s();
    group_sync<NT>();
    const float z2 = quad_dot<R, M2, W == 8 ? 16 : 32>(w2, s_h1, at_part) + b2;
    lds_ref(s_h2, at_row) = tanh32(z2);
    if (S::kShared && is_as) s_as[srow] = a_times_s();
    group_sync<NT>();
    if (is_last) {
      // inputs SL s + i of slice s, at place (i mod 4, SL s / 4 + i / 4)
      float h2[SL];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        typedef float run __attribute__((ext_vector_type(SL / 4)));
        const run v = lds_at<run>(s_h2 + c * P, at_slice);
#pragma unroll
        for (int i = 0; i < SL / 4; ++i) h2[4 * i + c] = v[i];
      }
      float pa = 0.0f;
#pragma unroll
      for (int i = 0; i < SL; ++i) pa = fma32(aux[S::kAuxW3 + i], h2[i], pa);
      pa = slice_fold_sum(pa);
      const float a = tanh32(pa + aux[S::kAuxB3]);             // action lane mod 8
      if (is_out && lane < A) s_ra[slot][lane] = a;
      // every row of 16 lanes holds all the actions, action k in its lane k
      float ak[A], ba = 0.0f;
      row_bcast8(a, ak);
#pragma unroll
      for (int k = 0; k < A; ++k) ba = fma32(aux[S::kAuxB + k], ak[k], ba);
      if (S::kShared) as = s_as[srow];
      const float sn = tanh32(as + ba);
      if (dyn_lane) lds_ref(s_x, at_srow) = sn;
      // lane 0 holds component 0 of the new state
      failed = p.death_mode != 0 &&
               __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(sn), 0)) < p.death_below;
      if (failed) {
        if (S::kShared && lane == 0) *s_fail = 1;
      } else if (is_out && dyn_lane && srow <= 4) {
        s_rs[srow][slot] = sn;
      }
    }
    if (S::kShared) {
      __syncthreads();
      read_state();
      failed = *s_fail != 0;   // the same value in every thread after the barrier
    } else {
      wave_sync();
      read_state();
    }
    if (failed) break;
    ++valid;
    // a full ring: the output wave, its only writer, folds it in
    if ((valid & (kRing - 1)) == 0 && is_out) flush_ring<A>(s_ra, s_rs, kRing, lane, acc);
  }
  if (!is_out || !mine) return;
  flush_ring<A>(s_ra, s_rs, valid & (kRing - 1), lane, acc);
  // death flag (Appendix A.4 i): a NaN objective is never inserted
  const bool dead = (p.death_mode == 2 && failed) || valid == 0;
  if (lane == 0) {
    p.off_fit[j] = dead ? __builtin_nanf("") : acc;
    p.off_par[2 * j] = q.c1;
    p.off_par[2 * j + 1] = q.c2;
    p.off_bank[j] = (uint8_t)q.banks;
    p.off_won[j] = 0;
  } else if (lane <= 4) {
    p.off_desc[(size_t)j * 4 + (lane - 1)] = valid > 0 ? acc / (float)valid : 0.0f;
  }
}

constexpr int rollout_waves(int hid) { return hid / 64; }

template <int H, bool GEN0, bool KEEP>
__global__ __launch_bounds__((RolloutShape<H, rollout_waves(H)>::kThreads),
                             (RolloutShape<H, rollout_waves(H)>::kWavesPerSimd))
void k_rollout(const Params p, uint32_t g) {
  rollout<H, rollout_waves(H), GEN0, KEEP>(p, g);
}

// The 128-wide policies of a batch of at most one individual per CU.
template <bool GEN0, bool KEEP>
__global__ __launch_bounds__((RolloutShape<128, 8>::kThreads), (RolloutShape<128, 8>::kWavesPerSimd))
void k_rollout_few(const Params p, uint32_t g) {
  rollout<128, 8, GEN0, KEEP>(p, g);
}

// Winners of a policy batch: a workgroup takes kRegenCellsMlp consecutive
// cells and, for each whose key names an offspring, all 256 threads write
// that offspring's genotype (same gene formula as the rollout's prologue) into
// the cell's other bank -- policy rows are long, so one row is spread over the
// whole workgroup.  After a barrier the cells record objective and descriptor,
// switch bank and take the incumbent key.
constexpr int kRegenCellsMlp = 8;

template <bool GEN0>
__global__ __launch_bounds__(256) void k_regen_mlp(const Params p, uint32_t g) {
  if (blockIdx.x == gridDim.x - 1) {
    compact_filled(p);
    return;
  }
  const int tid = threadIdx.x;
  const int first = blockIdx.x * kRegenCellsMlp;
  const int nblk = (p.n + 3) >> 2;
  __shared__ uint64_t s_key[kRegenCellsMlp];
  __shared__ float4 s_ntab[kNormalRows];
  if (!stage_keys<kRegenCellsMlp>(p, first, s_key)) return;
  if (!GEN0) {
    stage_normal_table(s_ntab, p.ntab, tid, 256);
    __syncthreads();
  }
  const Tables tb{s_ntab};
  for (int t = 0; t < kRegenCellsMlp; ++t) {
    const uint64_t key = s_key[t];
    if (!names_offspring(key)) continue;
    const int c = first + t;
    const int j = p.nb - 1 - (int)(uint32_t)key;
    Pair q{nullptr, nullptr, 0.0f, -1, -1, 0u};
    if (!GEN0) q = recorded_pair(p, g, j, tb);
    float* dst = geno_row(p, p.arch_slot[c] ^ 1u, c);
    for (int blk = tid; blk < nblk; blk += 256)
      *reinterpret_cast<float4*>(dst + 4 * blk) = mlp_gene_block<GEN0>(p, q, g, j, blk);
  }
  __syncthreads();
  if (tid < kRegenCellsMlp) {
    const uint64_t key = s_key[tid];
    if (names_offspring(key)) finish_winner(p, first + tid, p.nb - 1 - (int)(uint32_t)key, key);
  }
}

// Launchers: `go(kernel, grid, block, args...)` makes the launch.
// Waves per individual.  64 wide: one (two or four shorten the layers by less
// than their barriers cost: 230 and 199 us against 200 us for 64 to 256
// individuals and 250 steps, 239 and 340 us against 239 us for 1024).  128
// wide: two, whose weights leave room for two waves per SIMD, or eight of one
// row per quad while there is at most one individual per CU (64 to 256
// individuals, 400 steps: 391 us against 436 us; 512: 590 against 470 us).
constexpr int kEightWaveBatch = 256;

template <int H, class Go>
inline void launch_rollout_as(const Params& p, bool gen0, uint32_t g, bool keep, const Go& go) {
  using S = RolloutShape<H, rollout_waves(H)>;
  const dim3 grid(((unsigned)p.nb + S::kInd - 1u) / S::kInd), block(S::kThreads);
  if (gen0) {
    if (keep) go(k_rollout<H, true, true>, grid, block, p, g);
    else go(k_rollout<H, true, false>, grid, block, p, g);
  } else {
    if (keep) go(k_rollout<H, false, true>, grid, block, p, g);
    else go(k_rollout<H, false, false>, grid, block, p, g);
  }
}

template <class Go>
inline void launch_rollout(const Params& p, bool gen0, uint32_t g, bool keep, const Go& go) {
  if (p.hid == 64) {
    launch_rollout_as<64>(p, gen0, g, keep, go);
  } else if (p.nb > kEightWaveBatch) {
    launch_rollout_as<128>(p, gen0, g, keep, go);
  } else {
    const dim3 grid((unsigned)p.nb), block(RolloutShape<128, 8>::kThreads);
    if (gen0) {
      if (keep) go(k_rollout_few<true, true>, grid, block, p, g);
      else go(k_rollout_few<true, false>, grid, block, p, g);
    } else {
      if (keep) go(k_rollout_few<false, true>, grid, block, p, g);
      else go(k_rollout_few<false, false>, grid, block, p, g);
    }
  }
}

template <class Go>
inline void launch_mlp_regen(const Params& p, bool gen0, uint32_t g, const Go& go) {
  const dim3 grid(regen_blocks(p.C, kRegenCellsMlp)), block(256);
  if (gen0) go(k_regen_mlp<true>, grid, block, p, g);
  else go(k_regen_mlp<false>, grid, block, p, g);
}

}  // namespace qd
