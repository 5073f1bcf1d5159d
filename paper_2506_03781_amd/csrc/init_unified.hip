// Unified initialisation of UniQuan_F's parameters (Sec. 3 "Unified
// initialization"; appendix algorithms "Unified Initialization" and "General
// alternating update"; appendix "Details of clipping strategies").
//
// Per group of g weights: a grid search over gamma = j/G of candidate
// (Delta', z'_U) from a clipping strategy; for each, wbar = T_F(w) with
// s = s_r = 1, the general alternating update (greedy start, then T rounds of
// least-squares alpha, nearest codes and, with a one-point grid, the mean
// shift z_B), and the error ||w - Q*(w)||^2; the first smallest error wins.
//
// Mapping: each lane holds 8 consecutive weights, a group is g/8 adjacent
// lanes, a wavefront 512 weights.  Everything stays in registers except each
// group's 2^k-level table (LDS, wave-private).  The arithmetic follows one
// fixed order so that every code and every scale is reproducible:
//   * group sums are pairwise with adjacent pairing: a lane's 8 values as
//     ((v0+v1)+(v2+v3))+((v4+v5)+(v6+v7)), then xor-butterflies over lane
//     distance 1, 2, 4, ... (each step adds the sibling subtree);
//   * C^T C holds integers; its inverse is exact: alpha_a =
//     fp32( fp64(sum_b adj_ab v_b) / det ) with the integer adjugate, where
//     every product adj_ab v_b is exact in fp64 (C^T C and its adjugate are
//     positive semidefinite, so |adj_ab| <= g^3 <= 2^27, and v is fp32);
//     det = 0 keeps the previous alpha; where a group has at least
//     k (k + 1) / 2 lanes, each of its lanes computes one distinct adjugate
//     entry and lane a forms alpha_a (shuffles gather the operands), instead
//     of every lane solving the whole system;
//   * nearest level: first minimum of |fl(wbar - q)| over the ascending table
//     (the forward's rule), a constant group takes Delta' = 1.
// ALU-bound: the weights are read once and stay in registers for all G * T
// rounds.
#include "uq_device.h"
#include "uq_launch.h"

namespace uq {

struct InitArgs {
  int64_t N;
  int logg, gpr, G, T, clip;
  const void* W;
  float* delta;
  float* z_u;
  float* alpha;
  float* z_b;
  uint8_t* codes;
  float* err;
  float* s;
  float* s_r;
};

// Value of the lane whose subtree is the sibling of this lane's at butterfly
// level M (lane distance M).  Levels 1 and 2 pair lanes by xor (quad_perm);
// from level 4 on every lane of a subtree holds the same partial sum, so the
// mirror patterns (lane i <-> 7-i within 8, 15-i within 16) reach the sibling
// subtree as xor would, without going through LDS.
template <int M>
__device__ __forceinline__ int sibling(int v) {
  if constexpr (M == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
  else if constexpr (M == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, false);  // quad_perm [2,3,0,1]
  else if constexpr (M == 4) return __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, false); // row_half_mirror
  else if constexpr (M == 8) return __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, false); // row_mirror
  else if constexpr (M == 16) return __builtin_amdgcn_ds_swizzle(v, 0x401F);             // lane ^ 16
  else return __shfl_xor(v, 32, 64);
}

template <int M>
__device__ __forceinline__ float sibling(float v) {
  return __builtin_bit_cast(float, sibling<M>(__builtin_bit_cast(int, v)));
}

// Butterfly over the LPG lanes of a group (sum, min or max).
template <int LPG, typename T, typename Op>
__device__ __forceinline__ T group_reduce(T t, Op op) {
  if constexpr (LPG >= 2) t = op(t, sibling<1>(t));
  if constexpr (LPG >= 4) t = op(t, sibling<2>(t));
  if constexpr (LPG >= 8) t = op(t, sibling<4>(t));
  if constexpr (LPG >= 16) t = op(t, sibling<8>(t));
  if constexpr (LPG >= 32) t = op(t, sibling<16>(t));
  if constexpr (LPG >= 64) t = op(t, sibling<32>(t));
  return t;
}

struct AddF { __device__ float operator()(float a, float b) const { return a + b; } };
struct AddI { __device__ int operator()(int a, int b) const { return a + b; } };
struct MinF { __device__ float operator()(float a, float b) const { return fminf(a, b); } };
struct MaxF { __device__ float operator()(float a, float b) const { return fmaxf(a, b); } };

// Pairwise sum over a group: the lane's 8 values, then lane distances 1, 2, ...
// (IEEE addition is commutative, so both lanes of a pair hold the same sum).
template <int LPG>
__device__ __forceinline__ float group_sum(const float (&v)[8]) {
  const float t = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
  return group_reduce<LPG>(t, AddF());
}

__device__ __forceinline__ uint32_t pack4(int c0, int c1, int c2, int c3) {
  return uint32_t(c0) | (uint32_t(c1) << 8) | (uint32_t(c2) << 16) | (uint32_t(c3) << 24);
}

// Signed minors of C^T C.  M is symmetric with |M_ab| <= g <= 512, so every
// factor fits 24 bits (2x2 minors < 2^19) and every product 32 bits: the
// full-rate 24-bit multiply is exact here.
__device__ __forceinline__ int det2(int a, int b, int c, int d) { return __mul24(a, d) - __mul24(b, c); }

template <int K>
__device__ __forceinline__ int cofactor(const int (&M)[K][K], int r, int c) {
  // (-1)^(r+c) det(M without row r and column c); r, c are compile-time after
  // unrolling, so the index maps resolve statically.
  int S[3][3];
#pragma unroll
  for (int i = 0, ii = 0; i < K; ++i) {
    if (i == r) continue;
#pragma unroll
    for (int j = 0, jj = 0; j < K; ++j) {
      if (j == c) continue;
      S[ii][jj] = M[i][j];
      ++jj;
    }
    ++ii;
  }
  int d;
  if constexpr (K == 2) {
    d = S[0][0];
  } else if constexpr (K == 3) {
    d = det2(S[0][0], S[0][1], S[1][0], S[1][1]);
  } else {
    d = __mul24(S[0][0], det2(S[1][1], S[1][2], S[2][1], S[2][2])) -
        __mul24(S[0][1], det2(S[1][0], S[1][2], S[2][0], S[2][2])) +
        __mul24(S[0][2], det2(S[1][0], S[1][1], S[2][0], S[2][1]));
  }
  return ((r + c) & 1) ? -d : d;
}

// alpha = (C^T C)^{-1} v with the exact inverse adj / det; unchanged if det = 0.
template <int K>
__device__ __forceinline__ void solve_alpha(const int (&M)[K][K], const float (&v)[K], float (&al)[K]) {
  int adj[K][K];
  if constexpr (K == 1) {
    adj[0][0] = 1;
  } else {
#pragma unroll
    for (int a = 0; a < K; ++a)
#pragma unroll
      for (int b = a; b < K; ++b) {
        adj[a][b] = cofactor<K>(M, b, a);  // adj of a symmetric matrix is symmetric
        adj[b][a] = adj[a][b];
      }
  }
  // Laplace along row 0; exact (|terms| < 2^40).  Every product below is
  // exact in fp64, so fma(p, q, S) equals S + p*q rounded once, as in the
  // ascending-b sum it implements.
  double det = 0.0;
#pragma unroll
  for (int b = 0; b < K; ++b) det = __builtin_fma(double(M[0][b]), double(adj[b][0]), det);
  if (det == 0.0) return;
#pragma unroll
  for (int a = 0; a < K; ++a) {
    double S = double(adj[a][0]) * double(v[0]);
#pragma unroll
    for (int b = 1; b < K; ++b) S = __builtin_fma(double(adj[a][b]), double(v[b]), S);
    al[a] = float(S / det);
  }
}

// The same solve spread over the LPG lanes of a group (LPG >= K (K + 1) / 2):
// lane j < K (K + 1) / 2 computes the j-th of the adjugate's distinct entries
// adj_ab, a <= b in row-major order (the cofactor of M without row b and
// column a, its rows and columns chosen by per-lane selects), lane a < K
// gathers row a of the adjugate and forms alpha_a with the arithmetic of
// solve_alpha, and every lane gathers the K results.  The determinant is the
// same row-0 expansion, so the results are those of solve_alpha.
template <int K>
__device__ __forceinline__ int pair_index(int a, int b) {  // a <= b
  return a * K - (a * (a - 1)) / 2 + (b - a);
}

// The minor of M for adjugate entry jl (its rows and columns picked by
// per-lane selects) and the parity of its cofactor's sign.
template <int K>
__device__ __forceinline__ int lane_minor(const int (&M)[K][K], int jl, int (&S)[3][3]) {
  // (a, b) of pair jl, 2 bits each, 4 bits per pair
  uint64_t tab = 0;
#pragma unroll
  for (int a = 0; a < K; ++a)
#pragma unroll
    for (int b = a; b < K; ++b) tab |= uint64_t(a | (b << 2)) << (4 * pair_index<K>(a, b));
  const int jc = jl < K * (K + 1) / 2 ? jl : 0;
  const int e = int(tab >> (4 * jc)) & 15;
  const int c = e & 3, r = e >> 2;  // the minor without row r = b and column c = a
  int R[3][K];
#pragma unroll
  for (int i = 0; i < K - 1; ++i)
#pragma unroll
    for (int j = 0; j < K; ++j) R[i][j] = i >= r ? M[i + 1][j] : M[i][j];
#pragma unroll
  for (int i = 0; i < K - 1; ++i)
#pragma unroll
    for (int j = 0; j < K - 1; ++j) S[i][j] = j >= c ? R[i][j + 1] : R[i][j];
  return (r + c) & 1;
}

template <int K>
__device__ __forceinline__ int lane_cofactor(const int (&M)[K][K], int jl) {
  if constexpr (K == 1) {
    return 1;
  } else {
    int S[3][3];
    const int odd = lane_minor<K>(M, jl, S);
    int d;
    if constexpr (K == 2) {
      d = S[0][0];
    } else if constexpr (K == 3) {
      d = det2(S[0][0], S[0][1], S[1][0], S[1][1]);
    } else {
      d = __mul24(S[0][0], det2(S[1][1], S[1][2], S[2][1], S[2][2])) -
          __mul24(S[0][1], det2(S[1][0], S[1][2], S[2][0], S[2][2])) +
          __mul24(S[0][2], det2(S[1][0], S[1][1], S[2][0], S[2][1]));
    }
    return odd ? -d : d;
  }
}

template <int K, int LPG>
__device__ __forceinline__ void solve_alpha_dist(const int (&M)[K][K], const float (&v)[K], float (&al)[K], int jl,
                                                 int lane) {
  static_assert(LPG >= K * (K + 1) / 2, "one adjugate entry per lane");
  const int mine = lane_cofactor<K>(M, jl);
  const int base = lane - jl;
  // column 0 of the adjugate, the same in every lane of the group
  double det = 0.0;
#pragma unroll
  for (int b = 0; b < K; ++b)
    det = __builtin_fma(double(M[0][b]), double(__shfl(mine, base + pair_index<K>(0, b), 64)), det);
  if (det == 0.0) return;
  // row jl of the adjugate (lanes jl >= K take row K - 1 and discard it)
  const int ar = jl < K ? jl : K - 1;
  double S = 0.0;
#pragma unroll
  for (int b = 0; b < K; ++b) {
    const int idx = ar <= b ? pair_index<K>(ar, b) : pair_index<K>(b, ar);
    const double t = double(__shfl(mine, base + idx, 64));
    S = b == 0 ? t * double(v[0]) : __builtin_fma(t, double(v[b]), S);
  }
  const float out = float(S / det);
#pragma unroll
  for (int a = 0; a < K; ++a) al[a] = __shfl(out, base + a, 64);
}

// Ascending level table of the lane's group in LDS (raw, sorted, code_of).
// jl = lane index within the group.
template <int K>
__device__ __forceinline__ void build_table(float* raw, float* qs, uint8_t* cof, const float (&al)[K], float zb,
                                            int jl, int lpg) {
  constexpr int L = 1 << K;
  for (int b = jl; b < L; b += lpg) {
    float q = zb;
#pragma unroll
    for (int i = 0; i < K; ++i) q = ((b >> i) & 1) ? q + al[i] : q - al[i];
    raw[b] = q;
  }
  wave_lds_sync();
  for (int b = jl; b < L; b += lpg) {
    const float q = raw[b];
    int rank = 0;
#pragma unroll
    for (int b2 = 0; b2 < L; ++b2) {
      const float q2 = raw[b2];
      rank += (q2 < q) | ((q2 == q) & (b2 < b));
    }
    qs[rank] = q;
    cof[rank] = uint8_t(b);
  }
  wave_lds_sync();
}

// ---------------------------------------------------------------------------
// The round's mapping step for groups with a lane per level (k > 1).
//
// The kernel is bound by vector issue (every cycle at four per instruction, by the
// counters of 4096 x 4096 at k = 4), so the step counts instructions.  Where neighbouring levels are separated by more than 2^-20 of
// any distance that can occur, their distances from a weight stay apart after
// rounding: there is no run of equal distances to walk back, and the nearest
// level is one of the two around the weight.  A level of -infinity in front
// and positions counted by add-with-carry leave 16 instructions and three LDS
// operations per weight (28 and seven with the general search).  The levels'
// order seldom changes between rounds: lane j evaluates the level of the code
// that was j-th last time, and only an order that fails the separation test is
// ranked again (16% of the calls at k = 4, g = 128).
//
// A weight's state between rounds is one word, read from a table by position:
// bits 31 .. 32-K the code's bits inverted (bit K-1 first, so a shift brings
// bit b's sign to bit 31), and at 4 n, for the n-th pair p < q of bits (row
// order), whether bits p and q differ: eight words added give the lane's
// disagreement counts of all pairs.
// 4096 x 4096, k = 4, g = 128, G = 30, T = 15: 9.1 ms, against 13.3 ms with the
// general table and search for every round.
// ---------------------------------------------------------------------------
template <int K>
__device__ __forceinline__ uint32_t code_word(int c) {
  uint32_t w = (uint32_t(~c) & ((1u << K) - 1u)) << (32 - K);
#pragma unroll
  for (int p = 0, n = 0; p < K; ++p)
#pragma unroll
    for (int q = p + 1; q < K; ++q, ++n) w |= uint32_t(((c >> p) ^ (c >> q)) & 1) << (4 * n);
  return w;
}

template <int K>
__device__ __forceinline__ uint32_t word_code(uint32_t w) {
  return (~w) >> (32 - K);
}

// x with the sign of code bit b (+ when set) of word w; xs holds x's own sign
// bit in every place (x's bits shifted right arithmetically by 31).
template <int K>
__device__ __forceinline__ float signed_by(float x, uint32_t wx, int b) {
  return __builtin_copysignf(x, __uint_as_float(wx << (K - 1 - b)));
}

__device__ __forceinline__ uint32_t sign_fill(float x) { return uint32_t(int(__float_as_uint(x)) >> 31); }

// One group's table in LDS: lv[1 + j] the level at position j, lv[0] =
// -infinity; words[1 + j] the word of its code.
struct StepTable {
  float* lv;
  uint32_t* words;
};

// Levels of the group at (al, zb) into the table.  jl: lane within the group
// (lanes past the last level only vote); myc: code at this lane's position,
// kept between calls; myq: its level; bound: at least |x| for every weight of
// the group; skip: lane outside the matrix.  Returns (the same in every lane)
// whether the levels of every group are well separated.
template <int K>
__device__ __forceinline__ bool step_table(const StepTable& t, const uint32_t* wordc, const float (&al)[K], float zb,
                                           int jl, int& myc, float& myq, float bound, bool skip) {
  constexpr int L = 1 << K;
  auto level = [&](int c) {
    float q = zb;
#pragma unroll
    for (int b = 0; b < K; ++b) q = ((c >> b) & 1) ? q + al[b] : q - al[b];
    return q;
  };
  const bool last = jl >= L - 1 || skip;
  // whether the next position's level (the next lane's: positions 0 .. L-1 lie
  // in one row of 16 lanes) is far enough above
  auto separated = [&](float q) {
    const float nb = __builtin_bit_cast(
        float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, q), 0x101, 0xF, 0xF, true));
    return __all((nb - q) > 0x1p-20f * (bound + fabsf(q)) || last) != 0;
  };
  float q = level(myc);
  bool ok = separated(q);
  if (!ok) {
    // rank the levels by (value, code): rank = levels below, counted as
    // q2 < q, or for smaller codes q2 < the float after q
    const int b = jl & (L - 1);
    const float r = level(b) + 0.0f;  // -0 becomes +0
    const float up = __uint_as_float(__float_as_uint(r) + ((int(__float_as_uint(r)) >> 31) | 1));
    if (jl < L) t.lv[1 + b] = r;
    wave_lds_sync();
    int rank = 0;
#pragma unroll
    for (int b2 = 0; b2 < L; ++b2) rank += t.lv[1 + b2] < (b2 < b ? up : r) ? 1 : 0;
    if (jl < L) t.words[1 + rank] = uint32_t(b);
    wave_lds_sync();
    myc = int(t.words[1 + b]) & (L - 1);
    wave_lds_sync();
    if (jl < L) t.words[1 + b] = wordc[myc];
    q = level(myc);
    ok = separated(q);
  }
  myq = q;
  if (jl < L) t.lv[1 + jl] = q;
  wave_lds_sync();
  return ok;
}

// pos = 2 pos + (x >= t)
__device__ __forceinline__ void shift_in(int& pos, float x, float t) {
  asm("v_cmp_ge_f32_e32 vcc, %1, %2\n\tv_addc_co_u32_e32 %0, vcc, %0, %0, vcc" : "+v"(pos) : "v"(x), "v"(t) : "vcc");
}

// The words of N weights x(i): the levels at or below x among all but the last
// counted by bisection (its first two steps from registers), then the nearer
// of the two levels around x, the lower one on equal distances.
template <int K, int N, typename X, typename Put>
__device__ __forceinline__ void map_words(const StepTable& t, bool ok, const X& x, const Put& put) {
  constexpr int L = 1 << K;
  if (ok) {
    const float* q = t.lv + 1;
    const float tm = q[L / 2 - 1], tlo = q[K > 1 ? L / 4 - 1 : 0], thi = q[K > 1 ? 3 * L / 4 - 1 : 0];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float xi = x(i);
      int pos = 0;
      if constexpr (K == 1) {
        shift_in(pos, xi, tm);
      } else {
        float t2;
        asm("v_cmp_ge_f32_e32 vcc, %2, %3\n\t"
            "v_cndmask_b32_e32 %1, %4, %5, vcc\n\t"
            "v_cndmask_b32_e64 %0, 0, 1, vcc\n\t"
            "v_cmp_ge_f32_e32 vcc, %2, %1\n\t"
            "v_addc_co_u32_e32 %0, vcc, %0, %0, vcc"
            : "=&v"(pos), "=&v"(t2)
            : "v"(xi), "v"(tm), "v"(tlo), "v"(thi)
            : "vcc");
        if constexpr (K == 4) shift_in(pos, xi, q[4 * pos + 1]);
        if constexpr (K >= 3) shift_in(pos, xi, q[2 * pos]);
      }
      const float da = xi - t.lv[pos], db = xi - t.lv[pos + 1];
      asm("v_cmp_lt_f32_e64 vcc, |%1|, |%2|\n\tv_addc_co_u32_e32 %0, vcc, 0, %0, vcc"
          : "+v"(pos)
          : "v"(db), "v"(da)
          : "vcc");
      put(i, t.words[pos]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      float dist;
      put(i, t.words[1 + nearest_full_k<K>(t.lv + 1, x(i), dist)]);
    }
  }
}

// Mapping by thresholds for groups with a lane per level; two levels (k = 1) are found
// as fast without (2048 x 4096, g = 128, one grid point: 65 us with it, 59 without; 30: equal).
__host__ __device__ constexpr bool init_step(int logg, int k) { return k > 1 && logg - 3 >= k; }

// A wavefront's tables: of L + 1 levels and words a group, or raw and sorted
// levels and codes.  The second set the number of workgroups a CU holds for small
// groups (k = 4, g = 8: 37 KB each, four of them).
__host__ __device__ constexpr size_t init_wave_lds_bytes(int logg, int k) {
  const size_t groups = size_t(512) >> logg, e = groups << k;
  return init_step(logg, k) ? (8 * (e + groups) + 15) & ~size_t(15) : (e * 9 + 15) & ~size_t(15);
}
static_assert(4 * init_wave_lds_bytes(3, 4) <= 36 * 1024, "four workgroups a CU at k = 4, g = 8");

template <int WDT, int K, int LOGG>
__global__ __launch_bounds__(kThreads) void init_unified_kernel(InitArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  __shared__ uint32_t wordc[1 << K];
  constexpr int L = 1 << K;
  constexpr int lpg = 1 << (LOGG - 3);  // lanes per group
  constexpr bool kStep = init_step(LOGG, K);
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int jl = lane & (lpg - 1);
  if constexpr (kStep) {
    if (threadIdx.x < L) wordc[threadIdx.x] = code_word<K>(threadIdx.x);
    __syncthreads();
  }
  const int64_t wave_off = (int64_t(blockIdx.x) * (kThreads / 64) + wave) * 512;
  if (wave_off >= a.N) return;  // whole wavefront past the end (no block barriers below)
  const int64_t off = wave_off + lane * 8;
  const bool active = off < a.N;
  const int64_t gid = active ? (off >> LOGG) : 0;

  // This group's table in the wave's LDS region.
  char* wbase = smem + size_t(wave) * init_wave_lds_bytes(LOGG, K);
  const int gl = lane / lpg;  // group index within the wave
  const int gpw = 64 / lpg;
  float* raw = reinterpret_cast<float*>(wbase) + gl * L;
  float* qs = reinterpret_cast<float*>(wbase) + (gpw + gl) * L;
  uint8_t* cof = reinterpret_cast<uint8_t*>(wbase) + size_t(2 * gpw * L) * 4 + gl * L;
  const StepTable tab{reinterpret_cast<float*>(wbase) + gl * (L + 1),
                      reinterpret_cast<uint32_t*>(wbase) + (gpw + gl) * (L + 1)};
  int myc = jl & (L - 1);
  float myq = 0.0f;
  if constexpr (kStep) {
    if (jl < L) tab.words[1 + jl] = wordc[jl];
    if (jl == 0) tab.lv[0] = -INFINITY;
  }

  float w[8];
  if (active) {
    load8<WDT>(a.W, off, w);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) w[i] = 0.0f;
  }
  float wm = w[0], wM = w[0];
#pragma unroll
  for (int i = 1; i < 8; ++i) {
    wm = fminf(wm, w[i]);
    wM = fmaxf(wM, w[i]);
  }
  wm = group_reduce<lpg>(wm, MinF());
  wM = group_reduce<lpg>(wM, MaxF());

  const float L1 = float(L - 1);
  const float zb0 = L1 * 0.5f;
  constexpr float inv_g = 1.0f / float(1 << LOGG);  // exact power of two
  constexpr int g = 1 << LOGG;

  float best_d = 1.0f, best_zu = 0.0f, best_zb = zb0, best_e = 0.0f, best_al[K];
  uint32_t best_c0 = 0, best_c1 = 0;
#pragma unroll
  for (int b = 0; b < K; ++b) best_al[b] = 0.0f;

  for (int j = 1; j <= a.G; ++j) {
    const float gamma = float(j) / float(a.G);
    float dl = (gamma * (wM - wm)) / L1;
    if (!(dl > 0.0f)) dl = 1.0f;
    float zu;
    if (a.clip == 0) zu = -(wm / dl);
    else if (a.clip == 1) zu = L1 - (wM / dl);
    else zu = -((gamma * wm) / dl);

    float wbar[8], x[8];
    float zb = zb0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      wbar[i] = (w[i] / dl) + zu;
      x[i] = wbar[i] - zb;
    }

    // Greedy start: one bit at a time.
    float al[K];
    int code[8];
    {
      float r[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        r[i] = x[i];
        code[i] = 0;
      }
#pragma unroll
      for (int b = 0; b < K; ++b) {
        float ab[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) ab[i] = fabsf(r[i]);
        const float ai = group_sum<lpg>(ab) * inv_g;
        al[b] = ai;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const bool plus = r[i] >= 0.0f;
          code[i] |= int(plus) << b;
          r[i] = plus ? r[i] - ai : r[i] + ai;
        }
      }
    }

    float e2[8];
    uint32_t c0 = 0, c1 = 0;
    if constexpr (kStep) {
      uint32_t wd[8], xs[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        wd[i] = wordc[code[i]];
        xs[i] = sign_fill(x[i]);
      }
      const float bound = fmaxf(fabsf((wm / dl) + zu), fabsf((wM / dl) + zu));
      for (int t = 0; t < a.T; ++t) {
        // alpha <- (C^T C)^{-1} C^T (wbar - z_B)
        float v[K];
        {
          uint32_t wx[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) wx[i] = wd[i] ^ xs[i];
#pragma unroll
          for (int b = 0; b < K; ++b) {
            float sx[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) sx[i] = signed_by<K>(x[i], wx[i], b);
            v[b] = group_sum<lpg>(sx);
          }
        }
        int M[K][K];
        M[0][0] = g;
        if constexpr (K > 1) {
          // the lane's counts (4-bit fields, at most 8), then in 8-bit fields
          // over 16 lanes (at most 128), the rest one by one
          uint32_t sum = wd[0];
#pragma unroll
          for (int i = 1; i < 8; ++i) sum += wd[i];
          int ev = int(sum & 0x000F0F0Fu), od = int((sum >> 4) & 0x000F0F0Fu);
          constexpr int kRow = lpg < 16 ? lpg : 16;
          ev = group_reduce<kRow>(ev, AddI());
          if constexpr (K > 2) od = group_reduce<kRow>(od, AddI());
#pragma unroll
          for (int p = 0, n = 0; p < K; ++p) {
            M[p][p] = g;
#pragma unroll
            for (int q = p + 1; q < K; ++q, ++n) {
              int dis = (((n & 1) ? od : ev) >> (8 * (n >> 1))) & 0xFF;
              if constexpr (lpg >= 32) dis += sibling<16>(dis);
              if constexpr (lpg >= 64) dis += sibling<32>(dis);
              M[p][q] = g - 2 * dis;
              M[q][p] = M[p][q];
            }
          }
        }
        if constexpr (lpg >= K * (K + 1) / 2) solve_alpha_dist<K, lpg>(M, v, al, jl, lane);
        else solve_alpha<K>(M, v, al);

        // C <- nearest level's code
        const bool ok = step_table<K>(tab, wordc, al, zb, jl, myc, myq, bound, !active);
        uint32_t diff = 0;
        map_words<K, 8>(tab, ok, [&](int i) { return wbar[i]; },
                        [&](int i, uint32_t nw) {
                          diff |= nw ^ wd[i];
                          wd[i] = nw;
                        });

        // z_B <- mean(wbar - C alpha), only with a one-point grid
        const float zb_prev = zb;
        if (a.G == 1) {
          float dd[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            float ca = 0.0f;
            const uint32_t cd = word_code<K>(wd[i]);
#pragma unroll
            for (int b = 0; b < K; ++b) ca = ((cd >> b) & 1u) ? ca + al[b] : ca - al[b];
            dd[i] = wbar[i] - ca;
          }
          zb = group_sum<lpg>(dd) * inv_g;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            x[i] = wbar[i] - zb;
            xs[i] = sign_fill(x[i]);
          }
        }

        // Unchanged codes and shift make this state a fixed point of the round
        // (the round is a deterministic function of C, z_B and, for a singular
        // C^T C, alpha), so the remaining rounds would reproduce it exactly.
        if (__all((diff == 0 && zb == zb_prev) || !active)) break;
      }

      // Candidate error ||w - Q*(w)||^2 with the forward's FULL mapping: the
      // last round's codes, unless z_B moved after them or there was no round.
      if (a.G == 1 || a.T == 0) {
        const bool ok = step_table<K>(tab, wordc, al, zb, jl, myc, myq, bound, !active);
        map_words<K, 8>(tab, ok, [&](int i) { return wbar[i]; }, [&](int i, uint32_t nw) { wd[i] = nw; });
      }
      if (jl < L) tab.lv[1 + myc] = myq;  // levels by code
      wave_lds_sync();
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint32_t cb = word_code<K>(wd[i]);
        if (i < 4) c0 |= cb << (8 * i);
        else c1 |= cb << (8 * (i - 4));
        const float what = dl * (tab.lv[1 + cb] - zu);
        const float d = w[i] - what;
        e2[i] = d * d;
      }
    } else {
      // Codes packed 4 per word: the C^T C counts and the fixed-point test use them.
      uint32_t cw0 = pack4(code[0], code[1], code[2], code[3]);
      uint32_t cw1 = pack4(code[4], code[5], code[6], code[7]);
      for (int t = 0; t < a.T; ++t) {
        // alpha <- (C^T C)^{-1} C^T (wbar - z_B)
        float v[K];
#pragma unroll
        for (int b = 0; b < K; ++b) {
          float sx[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) sx[i] = ((code[i] >> b) & 1) ? x[i] : -x[i];
          v[b] = group_sum<lpg>(sx);
        }
        int M[K][K];
        {
          // bit b of the lane's 8 codes, one bit per byte
          uint32_t p0[K], p1[K];
#pragma unroll
          for (int b = 0; b < K; ++b) {
            p0[b] = (cw0 >> b) & 0x01010101u;
            p1[b] = (cw1 >> b) & 0x01010101u;
          }
#pragma unroll
          for (int p = 0; p < K; ++p) {
            M[p][p] = g;
#pragma unroll
            for (int q = p + 1; q < K; ++q) {
              const int dis = __builtin_popcount(p0[p] ^ p0[q]) + __builtin_popcount(p1[p] ^ p1[q]);
              M[p][q] = g - 2 * group_reduce<lpg>(dis, AddI());
              M[q][p] = M[p][q];
            }
          }
        }
        if constexpr (lpg >= K * (K + 1) / 2) solve_alpha_dist<K, lpg>(M, v, al, jl, lane);
        else solve_alpha<K>(M, v, al);

        // C <- nearest level's code
        build_table<K>(raw, qs, cof, al, zb, jl, lpg);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          float dist;
          code[i] = cof[nearest_full_k<K>(qs, wbar[i], dist)];
        }
        const uint32_t nw0 = pack4(code[0], code[1], code[2], code[3]);
        const uint32_t nw1 = pack4(code[4], code[5], code[6], code[7]);

        // z_B <- mean(wbar - C alpha), only with a one-point grid
        const float zb_prev = zb;
        if (a.G == 1) {
          float dd[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            float ca = 0.0f;
#pragma unroll
            for (int b = 0; b < K; ++b) ca = ((code[i] >> b) & 1) ? ca + al[b] : ca - al[b];
            dd[i] = wbar[i] - ca;
          }
          zb = group_sum<lpg>(dd) * inv_g;
#pragma unroll
          for (int i = 0; i < 8; ++i) x[i] = wbar[i] - zb;
        }

        // Unchanged codes and shift make this state a fixed point of the round
        // (the round is a deterministic function of C, z_B and, for a singular
        // C^T C, alpha), so the remaining rounds would reproduce it exactly.
        const bool same = (nw0 == cw0) & (nw1 == cw1) & (zb == zb_prev);
        cw0 = nw0;
        cw1 = nw1;
        if (__all(same || !active)) break;
      }

      // Candidate error ||w - Q*(w)||^2 with the forward's FULL mapping.
      build_table<K>(raw, qs, cof, al, zb, jl, lpg);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float dist;
        const int pos = nearest_full_k<K>(qs, wbar[i], dist);
        const uint32_t cb = cof[pos];
        if (i < 4) c0 |= cb << (8 * i);
        else c1 |= cb << (8 * (i - 4));
        const float what = dl * (qs[pos] - zu);
        const float d = w[i] - what;
        e2[i] = d * d;
      }
    }
    const float e = group_sum<lpg>(e2);
    if (j == 1 || e < best_e) {
      best_e = e;
      best_d = dl;
      best_zu = zu;
      best_zb = zb;
#pragma unroll
      for (int b = 0; b < K; ++b) best_al[b] = al[b];
      best_c0 = c0;
      best_c1 = c1;
    }
  }

  if (!active) return;
  if (a.codes) store8u8(a.codes, off, make_uint2(best_c0, best_c1));
  if (a.s) {
    const float one[8] = {1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f};
    store8f(a.s, off, one);
  }
  if (jl == 0) {
    a.delta[gid] = best_d;
    a.z_u[gid] = best_zu;
    a.z_b[gid] = best_zb;
#pragma unroll
    for (int b = 0; b < K; ++b) a.alpha[gid * K + b] = best_al[b];
    if (a.err) a.err[gid] = best_e;
    if (a.s_r && (gid % a.gpr) == 0) a.s_r[gid / a.gpr] = 1.0f;
  }
}

// ---------------------------------------------------------------------------
// Groups of more than 512 weights (a whole row per group, up to 16384): one
// workgroup per group, NW wavefronts, lane l holding the E consecutive
// elements l E .. l E + E - 1 of the group zero-padded to P = 64 NW E (the
// next power of two; E >= 8), so the pairwise tree over the padded group is
// the lane's own pairwise sum of its E values, then the butterfly over the 64
// lanes of a wavefront, then the wavefronts' sums pairwise in order.  The
// weights, their transforms and the codes stay in registers; each wavefront
// keeps its own copy of the level table in LDS.  C^T C entries reach g, so
// its adjugate (|adj| <= g^3 < 2^42) and determinant are int64, exactly
// converted (the determinant rounded) to fp64, and the products adj_ab v_b
// round in fp64 and are added in ascending b, as written.
//
// With 16 wavefronts and one workgroup per CU the round was bound by its
// barriers (six: three reductions of two each).  A round now has one exchange
// with one barrier: the sums, the disagreement counts and whether the round
// before changed anything travel together (a fixed point is then seen one
// exchange later, with the same state), and two buffers alternate.  With the
// mapping step above, 1024 rows of 11008 at k = 3, G = 30, T = 15: 7.3 ms
// against 15.6.
// ---------------------------------------------------------------------------
// Pairwise sum of E values produced in index order (adjacent pairing): a
// stack of partial sums, one per level.
template <int E>
struct LaneTree {
  static constexpr int LG = __builtin_ctz(E);
  float st[LG + 1];
  template <int I>
  __device__ __forceinline__ void push(float v) {
#pragma unroll
    for (int l = 0; l < LG; ++l) {
      if (((I >> l) & 1) == 0) {
        st[l] = v;
        return;
      }
      v = st[l] + v;
    }
    st[LG] = v;
  }
};

template <int E, int I = 0, typename F>
__device__ __forceinline__ void tree_push_all(LaneTree<E>& t, const F& f) {
  if constexpr (I < E) {
    t.template push<I>(f(I));
    tree_push_all<E, I + 1>(t, f);
  }
}

// Exchange between the NW wavefronts of a workgroup of NF floats and NI
// integers, each already summed over the wavefront's lanes: pairwise sums of
// the floats in wavefront order and sums of the integers, in every lane.  Lane
// l reads wavefront l % NW's values and a butterfly over NW lanes adds them (a
// pairwise tree in order).  One barrier per exchange: the two buffers
// alternate, and a buffer is written again only after the barrier of the
// exchange in between, which every wavefront reaches after its reads.
template <int NW, int CAP>
struct Exchange {
  uint32_t (*buf)[NW][CAP];  // [2][NW][CAP] words in LDS
  int turn = 0;
  int lane, wave;
  template <int NF, int NI>
  __device__ __forceinline__ void sum(float (&f)[NF], int (&n)[NI]) {
    static_assert(NF + NI <= CAP, "exchange buffer too small");
    uint32_t(*b)[CAP] = buf[turn];
    turn ^= 1;
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < NF; ++i) b[wave][i] = __float_as_uint(f[i]);
#pragma unroll
      for (int i = 0; i < NI; ++i) b[wave][NF + i] = uint32_t(n[i]);
    }
    __syncthreads();
    const uint32_t* r = b[lane & (NW - 1)];
#pragma unroll
    for (int i = 0; i < NF; ++i) f[i] = group_reduce<NW>(__uint_as_float(r[i]), AddF());
#pragma unroll
    for (int i = 0; i < NI; ++i) n[i] = group_reduce<NW>(int(r[NF + i]), AddI());
  }
  // one float, already summed over a lane's values only
  __device__ __forceinline__ float lane_sum(float v) {
    float f[1] = {group_reduce<64>(v, AddF())};
    int none[1] = {0};
    sum(f, none);
    return f[0];
  }
};

// alpha = (C^T C)^{-1} v for C^T C entries up to 2^14, spread over the lanes
// of a wavefront as solve_alpha_dist: lane j < K (K + 1) / 2 computes one
// distinct adjugate entry in int64 (|adj| <= g^3 < 2^42), lane a < K forms
// alpha_a = (sum_b adj_ab v_b) / det with the exact int64 determinant (row-0
// expansion) converted to fp64 and the fp64 products added in ascending b,
// and every lane gathers the K results.  Unchanged if det = 0.
__device__ __forceinline__ int64_t shfl64(int64_t x, int src) {
  const int lo = __shfl(int(uint32_t(uint64_t(x))), src, 64);
  const int hi = __shfl(int(uint32_t(uint64_t(x) >> 32)), src, 64);
  return int64_t((uint64_t(uint32_t(hi)) << 32) | uint32_t(lo));
}

template <int K>
__device__ __forceinline__ void solve_alpha64_dist(const int (&M)[K][K], const float (&v)[K], float (&al)[K],
                                                   int lane) {
  int64_t mine = 1;
  if constexpr (K > 1) {
    int S0[3][3];
    const int odd = lane_minor<K>(M, lane, S0);
    int64_t S[3][3];
#pragma unroll
    for (int i = 0; i < K - 1; ++i)
#pragma unroll
      for (int j = 0; j < K - 1; ++j) S[i][j] = S0[i][j];
    int64_t d;
    if constexpr (K == 2) {
      d = S[0][0];
    } else if constexpr (K == 3) {
      d = S[0][0] * S[1][1] - S[0][1] * S[1][0];
    } else {
      d = S[0][0] * (S[1][1] * S[2][2] - S[1][2] * S[2][1]) - S[0][1] * (S[1][0] * S[2][2] - S[1][2] * S[2][0]) +
          S[0][2] * (S[1][0] * S[2][1] - S[1][1] * S[2][0]);
    }
    mine = odd ? -d : d;
  }
  int64_t det = 0;
#pragma unroll
  for (int b = 0; b < K; ++b) det += int64_t(M[0][b]) * shfl64(mine, pair_index<K>(0, b));
  if (det == 0) return;
  const double dd = double(det);
  const int ar = lane < K ? lane : K - 1;
  double S = 0.0;
#pragma unroll
  for (int b = 0; b < K; ++b) {
    const int idx = ar <= b ? pair_index<K>(ar, b) : pair_index<K>(b, ar);
    const double pr = double(shfl64(mine, idx)) * double(v[b]);
    S = b == 0 ? pr : S + pr;
  }
  const float out = float(S / dd);
#pragma unroll
  for (int a = 0; a < K; ++a) al[a] = __shfl(out, a, 64);
}

template <int WDT, int K, int NW, int E>
__global__ __launch_bounds__(NW * 64) void init_unified_big_kernel(InitArgs a, int g) {
  constexpr int L = 1 << K;
  constexpr int kCnt = (K * (K - 1) / 2 + 1) / 2;  // words of two 16-bit disagreement counts
  __shared__ float tab_lv[NW][L + 1];
  __shared__ uint32_t tab_words[NW][L + 1];
  __shared__ uint32_t wordc[L];
  __shared__ uint32_t xbuf[2][NW][8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t gid = blockIdx.x;
  const int64_t goff = gid * int64_t(g);
  const int e0 = int(threadIdx.x) * E;  // first padded element of this lane
  const StepTable tab{tab_lv[wave], tab_words[wave]};
  Exchange<NW, 8> ex{xbuf, 0, lane, wave};
  int myc = lane & (L - 1);
  float myq = 0.0f;
  if (threadIdx.x < L) wordc[threadIdx.x] = code_word<K>(threadIdx.x);
  if (lane < L) tab.words[1 + lane] = code_word<K>(lane);
  if (lane == 0) tab.lv[0] = -INFINITY;

  float w[E];
#pragma unroll
  for (int c = 0; c < E; c += 8) {
    float v[8];
    if (e0 + c < g) {
      load8<WDT>(a.W, goff + e0 + c, v);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = 0.0f;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) w[c + i] = v[i];
  }
  // validity: g is a multiple of 8, so chunks of 8 are whole
  uint32_t valid8 = 0;  // bit c/8: chunk c .. c+7 real
#pragma unroll
  for (int c = 0; c < E; c += 8)
    if (e0 + c < g) valid8 |= 1u << (c / 8);
#define UQ_VALID(i) (((valid8 >> ((i) / 8)) & 1u) != 0u)
  // A wavefront whose elements are all padding adds exact zeros to every sum:
  // it skips the per-element work and only joins the exchanges.  Padding
  // elements of a live wavefront keep x = 0 and word 0 (plus sign, no
  // disagreement), which add exact zeros too.
  const bool live = __builtin_amdgcn_readfirstlane(wave) * 64 * E < g;

  float wm = INFINITY, wM = -INFINITY;
#pragma unroll
  for (int i = 0; i < E; ++i)
    if (UQ_VALID(i)) {
      wm = fminf(wm, w[i]);
      wM = fmaxf(wM, w[i]);
    }
  wm = group_reduce<64>(wm, MinF());
  wM = group_reduce<64>(wM, MaxF());
  if (lane == 0) {
    xbuf[1][wave][0] = __float_as_uint(wm);
    xbuf[1][wave][1] = __float_as_uint(wM);
  }
  __syncthreads();
  wm = group_reduce<NW>(__uint_as_float(xbuf[1][lane & (NW - 1)][0]), MinF());
  wM = group_reduce<NW>(__uint_as_float(xbuf[1][lane & (NW - 1)][1]), MaxF());

  const float L1 = float(L - 1);
  const float zb0 = L1 * 0.5f;
  const float gf = float(g);
  float best_d = 1.0f, best_zu = 0.0f, best_zb = zb0, best_e = 0.0f, best_al[K];
  uint32_t best_cw[E / 4];  // codes packed four to a word
#pragma unroll
  for (int b = 0; b < K; ++b) best_al[b] = 0.0f;
#pragma unroll
  for (int q = 0; q < E / 4; ++q) best_cw[q] = 0u;

  for (int j = 1; j <= a.G; ++j) {
    const float gamma = float(j) / float(a.G);
    float dl = (gamma * (wM - wm)) / L1;
    if (!(dl > 0.0f)) dl = 1.0f;
    float zu;
    if (a.clip == 0) zu = -(wm / dl);
    else if (a.clip == 1) zu = L1 - (wM / dl);
    else zu = -((gamma * wm) / dl);
    const float bound = fmaxf(fabsf((wm / dl) + zu), fabsf((wM / dl) + zu));
    float wbar[E];
#pragma unroll
    for (int i = 0; i < E; ++i) wbar[i] = (w[i] / dl) + zu;
    float zb = zb0;

    // greedy start, one bit at a time
    float al[K];
    uint32_t wd[E];  // state words
    {
      float r[E];
      int code[E];
#pragma unroll
      for (int i = 0; i < E; ++i) {
        r[i] = UQ_VALID(i) ? wbar[i] - zb : 0.0f;
        code[i] = 0;
      }
#pragma unroll
      for (int b = 0; b < K; ++b) {
        float t = 0.0f;
        if (live) {
          LaneTree<E> tr;
          tree_push_all<E>(tr, [&](int i) { return UQ_VALID(i) ? fabsf(r[i]) : 0.0f; });
          t = tr.st[LaneTree<E>::LG];
        }
        const float ai = ex.lane_sum(t) / gf;
        if (live) {
#pragma unroll
          for (int i = 0; i < E; ++i) {
            const bool plus = r[i] >= 0.0f;
            code[i] |= int(plus) << b;
            r[i] = plus ? r[i] - ai : r[i] + ai;
          }
        }
        al[b] = ai;
      }
#pragma unroll
      for (int i = 0; i < E; ++i) wd[i] = UQ_VALID(i) ? wordc[code[i]] : 0u;
    }

    int same = 0;  // the previous round changed nothing in this wavefront
    for (int t = 0; t < a.T; ++t) {
      // C^T (wbar - z_B) and the disagreement counts of this wavefront
      float v[K];
      int cnt[kCnt + 1];
#pragma unroll
      for (int b = 0; b < K; ++b) v[b] = 0.0f;
#pragma unroll
      for (int q = 0; q <= kCnt; ++q) cnt[q] = 0;
      if (live) {
        float x[E];
        uint32_t wx[E];
#pragma unroll
        for (int i = 0; i < E; ++i) {
          x[i] = UQ_VALID(i) ? wbar[i] - zb : 0.0f;
          wx[i] = wd[i] ^ sign_fill(x[i]);
        }
#pragma unroll
        for (int b = 0; b < K; ++b) {
          LaneTree<E> tr;
          tree_push_all<E>(tr, [&](int i) { return signed_by<K>(x[i], wx[i], b); });
          v[b] = group_reduce<64>(tr.st[LaneTree<E>::LG], AddF());
        }
        if constexpr (K > 1) {
          // 4-bit fields over 8 weights, 8-bit ones over the lane and 4 lanes
          // (at most 64), 16-bit ones over the wavefront (at most 1024)
          int ev = 0, od = 0;
#pragma unroll
          for (int c = 0; c < E; c += 8) {
            uint32_t sum = wd[c];
#pragma unroll
            for (int i = 1; i < 8; ++i) sum += wd[c + i];
            ev += int(sum & 0x000F0F0Fu);
            od += int((sum >> 4) & 0x000F0F0Fu);
          }
          ev = group_reduce<4>(ev, AddI());
          od = group_reduce<4>(od, AddI());
          // pairs 2 q and 2 q + 1 in the halves of cnt[q]
#pragma unroll
          for (int q = 0; q < kCnt; ++q) {
            int c = ((ev >> (8 * q)) & 0xFF) | (((od >> (8 * q)) & 0xFF) << 16);
            c += sibling<4>(c);
            c += sibling<8>(c);
            c += sibling<16>(c);
            c += sibling<32>(c);
            cnt[q] = c;
          }
        }
      }
      // a wavefront of padding agrees with everything
      cnt[kCnt] = live ? same : int(t > 0);
      ex.sum(v, cnt);
      // Unchanged codes and shift in the whole group after the last round: a
      // fixed point, which the remaining rounds would reproduce exactly.
      if (cnt[kCnt] == NW) break;
      int M[K][K];
      M[0][0] = g;
      if constexpr (K > 1) {
#pragma unroll
        for (int p = 0, n = 0; p < K; ++p) {
          M[p][p] = g;
#pragma unroll
          for (int q = p + 1; q < K; ++q, ++n) {
            M[p][q] = g - 2 * ((cnt[n >> 1] >> (16 * (n & 1))) & 0xFFFF);
            M[q][p] = M[p][q];
          }
        }
      }
      solve_alpha64_dist<K>(M, v, al, lane);

      // C <- nearest level's code
      uint32_t diff = 0;
      if (live) {
        const bool ok = step_table<K>(tab, wordc, al, zb, lane, myc, myq, bound, false);
        map_words<K, E>(tab, ok, [&](int i) { return wbar[i]; },
                        [&](int i, uint32_t nw) {
                          nw = UQ_VALID(i) ? nw : 0u;
                          diff |= nw ^ wd[i];
                          wd[i] = nw;
                        });
      }
      const float zb_prev = zb;
      if (a.G == 1) {
        float tz = 0.0f;
        if (live) {
          LaneTree<E> tr;
          tree_push_all<E>(tr, [&](int i) {
            const uint32_t code = word_code<K>(wd[i]);
            float ca = 0.0f;
            for (int b = 0; b < K; ++b) ca = ((code >> b) & 1u) ? ca + al[b] : ca - al[b];
            return UQ_VALID(i) ? wbar[i] - ca : 0.0f;
          });
          tz = tr.st[LaneTree<E>::LG];
        }
        zb = ex.lane_sum(tz) / gf;
      }
      same = __all(diff == 0 && zb == zb_prev) ? 1 : 0;
    }

    // candidate error ||w - Q*(w)||^2 with the forward's FULL mapping: the
    // last round's codes, unless z_B moved after them or there was no round
    float te = 0.0f;
    if (live) {
      if (a.G == 1 || a.T == 0) {
        const bool ok = step_table<K>(tab, wordc, al, zb, lane, myc, myq, bound, false);
        map_words<K, E>(tab, ok, [&](int i) { return wbar[i]; },
                        [&](int i, uint32_t nw) { wd[i] = UQ_VALID(i) ? nw : 0u; });
      }
      if (lane < L) tab.lv[1 + myc] = myq;  // levels by code
      wave_lds_sync();
      LaneTree<E> tr;
      tree_push_all<E>(tr, [&](int i) {
        if (!UQ_VALID(i)) return 0.0f;
        const float what = dl * (tab.lv[1 + word_code<K>(wd[i])] - zu);
        const float d = w[i] - what;
        return d * d;
      });
      te = tr.st[LaneTree<E>::LG];
    }
    const float e = ex.lane_sum(te);
    if (j == 1 || e < best_e) {
      best_e = e;
      best_d = dl;
      best_zu = zu;
      best_zb = zb;
#pragma unroll
      for (int b = 0; b < K; ++b) best_al[b] = al[b];
#pragma unroll
      for (int q = 0; q < E / 4; ++q)
        best_cw[q] = pack4(word_code<K>(wd[4 * q]), word_code<K>(wd[4 * q + 1]), word_code<K>(wd[4 * q + 2]),
                           word_code<K>(wd[4 * q + 3]));
    }
  }

#pragma unroll
  for (int c = 0; c < E; c += 8) {
    if (e0 + c >= g) continue;
    if (a.codes) store8u8(a.codes, goff + e0 + c, make_uint2(best_cw[c / 4], best_cw[c / 4 + 1]));
    if (a.s) {
      const float one[8] = {1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f, 1.0f};
      store8f(a.s, goff + e0 + c, one);
    }
  }
#undef UQ_VALID
  if (threadIdx.x == 0) {
    a.delta[gid] = best_d;
    a.z_u[gid] = best_zu;
    a.z_b[gid] = best_zb;
#pragma unroll
    for (int b = 0; b < K; ++b) a.alpha[gid * K + b] = best_al[b];
    if (a.err) a.err[gid] = best_e;
    if (a.s_r && (gid % a.gpr) == 0) a.s_r[gid / a.gpr] = 1.0f;
  }
}

template <int WDT, int K>
static void launch_init_big(const InitArgs& a, int g, int64_t groups, hipStream_t st) {
  int p2 = 1024;
  while (p2 < g) p2 <<= 1;
  const dim3 grid(static_cast<unsigned>(groups));
  switch (p2) {
    case 1024: hipLaunchKernelGGL((init_unified_big_kernel<WDT, K, 2, 8>), grid, dim3(128), 0, st, a, g); break;
    case 2048: hipLaunchKernelGGL((init_unified_big_kernel<WDT, K, 4, 8>), grid, dim3(256), 0, st, a, g); break;
    case 4096: hipLaunchKernelGGL((init_unified_big_kernel<WDT, K, 4, 16>), grid, dim3(256), 0, st, a, g); break;
    case 8192: hipLaunchKernelGGL((init_unified_big_kernel<WDT, K, 8, 16>), grid, dim3(512), 0, st, a, g); break;
    default: hipLaunchKernelGGL((init_unified_big_kernel<WDT, K, 16, 16>), grid, dim3(1024), 0, st, a, g); break;
  }
}

template <int WDT>
static hipError_t launch_init_big_k(const InitArgs& a, int k, int g, int64_t groups, hipStream_t st) {
  switch (k) {
    case 1: launch_init_big<WDT, 1>(a, g, groups, st); break;
    case 2: launch_init_big<WDT, 2>(a, g, groups, st); break;
    case 3: launch_init_big<WDT, 3>(a, g, groups, st); break;
    default: launch_init_big<WDT, 4>(a, g, groups, st); break;
  }
  return hipGetLastError();
}

template <int WDT, int K>
static void launch_init_g(const InitArgs& a, dim3 grid, size_t lds, hipStream_t st) {
  switch (a.logg) {
    case 3: hipLaunchKernelGGL((init_unified_kernel<WDT, K, 3>), grid, dim3(kThreads), lds, st, a); break;
    case 4: hipLaunchKernelGGL((init_unified_kernel<WDT, K, 4>), grid, dim3(kThreads), lds, st, a); break;
    case 5: hipLaunchKernelGGL((init_unified_kernel<WDT, K, 5>), grid, dim3(kThreads), lds, st, a); break;
    case 6: hipLaunchKernelGGL((init_unified_kernel<WDT, K, 6>), grid, dim3(kThreads), lds, st, a); break;
    case 7: hipLaunchKernelGGL((init_unified_kernel<WDT, K, 7>), grid, dim3(kThreads), lds, st, a); break;
    case 8: hipLaunchKernelGGL((init_unified_kernel<WDT, K, 8>), grid, dim3(kThreads), lds, st, a); break;
    default: hipLaunchKernelGGL((init_unified_kernel<WDT, K, 9>), grid, dim3(kThreads), lds, st, a); break;
  }
}

template <int WDT>
static hipError_t launch_init_k(const InitArgs& a, int k, dim3 grid, size_t lds, hipStream_t st) {
  switch (k) {
    case 1: launch_init_g<WDT, 1>(a, grid, lds, st); break;
    case 2: launch_init_g<WDT, 2>(a, grid, lds, st); break;
    case 3: launch_init_g<WDT, 3>(a, grid, lds, st); break;
    default: launch_init_g<WDT, 4>(a, grid, lds, st); break;
  }
  return hipGetLastError();
}

hipError_t launch_init_unified(const InitUnifiedLaunch& p, hipStream_t st) {
  InitArgs a;
  a.N = p.R * p.C;
  a.logg = p.g > 512 ? 0 : __builtin_ctz(unsigned(p.g));
  a.gpr = int(p.C / p.g);
  a.G = p.grid_G;
  a.T = p.alt_T;
  a.clip = p.clip;
  a.W = p.W;
  a.delta = p.delta; a.z_u = p.z_u; a.alpha = p.alpha; a.z_b = p.z_b;
  a.codes = p.codes; a.err = p.err; a.s = p.s; a.s_r = p.s_r;
  if (p.g > 512) {
    const int64_t groups = a.N / p.g;
    if (p.w_dtype == BF16) return launch_init_big_k<BF16>(a, p.k, p.g, groups, st);
    return launch_init_big_k<F32>(a, p.k, p.g, groups, st);
  }
  const int64_t waves = (a.N + 511) / 512;
  const dim3 grid(unsigned((waves + 3) / 4));
  const size_t lds = 4 * init_wave_lds_bytes(a.logg, p.k);
  if (p.w_dtype == BF16) return launch_init_k<BF16>(a, p.k, grid, lds, st);
  return launch_init_k<F32>(a, p.k, grid, lds, st);
}

}  // namespace uq
