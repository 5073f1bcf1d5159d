// Deployment form of a folded layer (Theorem 1 output: codes C and
// Theta*_B = {alpha*, z*_B}) and the binary-coding product with a small
// batch of activations (the single inference step R_B(C; Theta*) of the
// table of quantization schemes).
//
// Stored form (g k + 16 (k + 1) bits per group, appendix "Memory usage"):
//   planes  uint32 [k][C/128][R][4]: word m of quad q of row r in plane i
//           holds bit i of the codes of columns 128 q + 32 m + j in bit j;
//   alpha16 fp16   [k][C/g][R], z16 fp16 [C/g][R] (round to nearest even).
// Rows are the fastest index of every array, so the 64 lanes of a wavefront
// that work on 64 consecutive rows read contiguous memory.
//
// Product Y[t][r] = sum_c X[t][c] What[r][c] with What = z* + sum_i alpha*_i
// sigma_i.  Per group, sum_c sigma_i x_c = 2 P_i - S with S the activation
// sum over the group and P_i the sum over the columns whose bit i is set, so
//   y = sum_groups [ sum_i (2 alpha*_i) P_i + (z* - sum_i alpha*_i) S ].
// P_i is gathered 4 columns at a time from per-workgroup lookup tables: for
// every 4-column nibble of the workgroup's column slab and every batch row,
// the 16 subset sums of those 4 activations.  One lookup replaces 4
// multiply-adds; the tables are built once per workgroup and shared by its
// 256 rows (one row per lane).  Slabs write fp32 partial rows that a second
// kernel sums in a fixed order (deterministic results).  Larger batches and
// small layers take the product on the matrix cores (bcq_mfma_kernel).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "uq_launch.h"

namespace uq {

// ---------------------------------------------------------------------------
// Packing
// ---------------------------------------------------------------------------
// Bit i of each of the four bytes of v, as a 4-bit number (byte b -> bit b):
// after masking, the bits sit at 0, 8, 16, 24; multiplying by
// 2^21 + 2^14 + 2^7 + 1 places byte b's bit at 21 + b and every other partial
// product at a distinct position outside 21..24, so no carries reach them.
__device__ __forceinline__ uint32_t gather_bit(uint32_t v, int i) {
  const uint32_t t = (v >> i) & 0x01010101u;
  return ((t * 0x00204081u) >> 21) & 0xFu;
}

// Blocks from nb2 on: one thread per (quad q, row r, word m), 32 code bytes ->
// one word per plane.  The others: alpha*, z*_B -> binary16, tiles of 64 rows x 16
// group columns turned in LDS so that reads run along a row's groups and writes
// along the rows (11008 x 4096, k = 3, g = 128: 13 us as a kernel of its own with a
// thread per parameter, whose reads were a row apart, after 12 for the planes; 13
// together here).
__global__ __launch_bounds__(256) void bcq_pack_kernel(const uint8_t* __restrict__ codes,
                                                       uint32_t* __restrict__ planes,
                                                       const float* __restrict__ alpha_star,
                                                       const float* __restrict__ z_star,
                                                       uint16_t* __restrict__ alpha16, uint16_t* __restrict__ z16,
                                                       int64_t R, int64_t C, int64_t gpr, int k, unsigned nb2) {
  constexpr int TR = 64, TJ = 16;
  __shared__ uint16_t t[5][TJ][TR + 2];  // k <= 4 scales and the offset
  if (blockIdx.x < nb2) {
    const uint32_t nj = uint32_t((gpr + TJ - 1) / TJ), rt = blockIdx.x / nj;
    const int64_t r0 = int64_t(rt) * TR, j0 = int64_t(blockIdx.x - rt * nj) * TJ;
    const int nr = int(min<int64_t>(TR, R - r0)), ng = int(min<int64_t>(TJ, gpr - j0));
    auto half = [](float v) { return __builtin_bit_cast(uint16_t, _Float16(v)); };
    // A lane per column (group, parameter) of 256 >> sh rows, U rows' loads in
    // flight, no division in the loops: these few workgroups are the launch's end
    // in a layer of 4096 x 4096 (an element a turn with two divisions: k = 4, g = 256
    // 9.2 us, the two launches before it 7.9, now 5.8).
    constexpr int U = 4;
    const float* ap = alpha_star + (r0 * gpr + j0) * k;  // 32-bit offsets from uniform bases: the tile's
    const float* zp = z_star + r0 * gpr + j0;            // rows span at most 2^23 elements
    const int rl = int(gpr) * k;
    const int per = ng * k, sh = per <= 16 ? 4 : per <= 32 ? 5 : 6, step = 256 >> sh;
    const int c = threadIdx.x & ((1 << sh) - 1);
    const int ca = k == 1 ? c : k == 2 ? c >> 1 : k == 3 ? (c * 43) >> 7 : c >> 2;  // c / k (c < 64)
    const int jz = threadIdx.x & (TJ - 1), rz = threadIdx.x / TJ;
    float z[TR * TJ / 256];
#pragma unroll
    for (int u = 0; u < TR * TJ / 256; ++u)
      z[u] = zp[min(rz + u * (256 / TJ), nr - 1) * int(gpr) + min(jz, ng - 1)];
    if (c < per)
      for (int r = threadIdx.x >> sh; r < nr; r += U * step) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = ap[min(r + u * step, nr - 1) * rl + c];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (r + u * step < nr) t[c - ca * k][ca][r + u * step] = half(v[u]);
      }
    if (jz < ng)
#pragma unroll
      for (int u = 0; u < TR * TJ / 256; ++u)
        if (rz + u * (256 / TJ) < nr) t[k][jz][rz + u * (256 / TJ)] = half(z[u]);
    __syncthreads();
    const int r = threadIdx.x & (TR - 1), w = __builtin_amdgcn_readfirstlane(threadIdx.x / TR);
    const bool few = ng < 256 / TR;  // the wavefronts share the arrays, else the groups
    if (r < nr)
      for (int i = few ? w : 0; i <= k; i += few ? 256 / TR : 1) {
        uint16_t* out = (i < k ? alpha16 + int64_t(i) * gpr * R : z16) + j0 * R + r0;
        for (int j = few ? 0 : w; j < ng; j += few ? 1 : 256 / TR) out[j * R + r] = t[i][j][r];
      }
    return;
  }
  const int64_t nq = C / 128;
  const uint32_t idx = (blockIdx.x - nb2) * 256 + threadIdx.x;  // below 2^32: a launch has no more threads
  if (idx >= nq * R * 4) return;
  const uint32_t m = idx & 3, rq = idx >> 2;  // q R + r
  const uint32_t q = rq / uint32_t(R);
  const int64_t r = rq - q * uint32_t(R);
  const uint4* src = reinterpret_cast<const uint4*>(codes + r * C + int64_t(q) * 128 + m * 32);
  const uint4 lo = src[0], hi = src[1];
  const uint32_t v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  for (int i = 0; i < k; ++i) {
    uint32_t word = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) word |= gather_bit(v[e], i) << (4 * e);
    planes[(int64_t(i) * nq * R + rq) * 4 + m] = word;
  }
}

hipError_t launch_bcq_pack(const BcqPackLaunch& p, hipStream_t st) {
  const int64_t nq = p.C / 128, gpr = p.C / p.g;
  const int64_t nb1 = (nq * p.R * 4 + 255) / 256, nb2 = ((p.R + 63) / 64) * ((gpr + 15) / 16);
  auto launch = [&](int64_t planes, int64_t params) {
    hipLaunchKernelGGL(bcq_pack_kernel, dim3(unsigned(planes + params)), dim3(256), 0, st, p.codes, p.planes,
                       p.alpha_star, p.z_star, p.alpha16, p.z16, p.R, p.C, gpr, p.k, unsigned(params));
  };
  if (nb1 + nb2 < (int64_t(1) << 24)) {
    launch(nb1, nb2);
  } else {  // a launch takes fewer than 2^32 threads
    launch(nb1, 0);
    launch(0, nb2);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Product
// ---------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct BcqArgs {
  const uint16_t* X;
  const uint32_t* planes;
  const uint16_t* alpha16;
  const uint16_t* z16;
  float* out;  // Y [T][R] (one slab) or partials [slabs][T][R]
  int64_t R, C, nq, gpr;
  int64_t rb0;       // first row block of this launch (MFMA kernel)
  int qps, qpg;      // quads per slab and per group
  uint32_t qpg_inv;  // ceil(2^32 / qpg): q / qpg = (q qpg_inv) >> 32 while q qpg < 2^32 (both at most 2^15)
};

// One v_bfe_u32 (the compiler otherwise splits a field extract of a masked
// word into a shift and an and).
template <int OFF>
__device__ __forceinline__ uint32_t byte_field(uint32_t w) {
  uint32_t r;
  asm volatile("v_bfe_u32 %0, %1, %2, 8" : "=v"(r) : "v"(w), "i"(OFF));
  return r;
}

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float(uint32_t(h) << 16); }
__device__ __forceinline__ float f16_to_f32(uint16_t h) { return float(__builtin_bit_cast(_Float16, h)); }

// Workgroup (bx, by): rows 256 bx .. 256 bx + 255 (one per lane), column
// quads QPS by .. QPS by + QPS - 1.  LDS: T tables of QPS * 32 nibbles x 16
// subset sums, then the T x QPS quad sums (activation sums S of the quads).
template <int K, int T, int QPS>
__global__ __launch_bounds__(256) void bcq_matmul_kernel(BcqArgs a) {
  constexpr int PER_T = QPS * 512;  // floats per batch row's tables
  __shared__ __attribute__((aligned(16))) float lut[T * PER_T + T * QPS];
  const int tid = threadIdx.x;
  const int64_t q0 = int64_t(blockIdx.y) * QPS;
  const int nqs = int(min<int64_t>(QPS, a.nq - q0));
  float* S = lut + T * PER_T;
  const int64_t r = int64_t(blockIdx.x) * 256 + tid;
  const bool live = r < a.R;

  // The activations this thread turns into tables (nibble tables e = tid +
  // 256 u of the T x nqs x 32 in the slab) are loaded first, then this lane's
  // plane words and parameters for the whole slab: loads complete in issue
  // order, so the table build waits only for the activations while the
  // plane loads stay in flight.
  constexpr int NT = (T * QPS * 32 + 255) / 256;  // nibble tables per thread (upper bound)
  constexpr int LOG_FULL = QPS == 4 ? 7 : QPS == 2 ? 6 : 5;  // log2(QPS * 32)
  const bool full = nqs == QPS;
  const int n_tab = T * nqs * 32;
  const uint16_t* xs = a.X + q0 * 128;
  uint2 xv[NT];
  // loads are unconditional (indices clamped into range) so that no branch
  // splits the load sequence; clamped values are never used
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int e = min(tid + 256 * u, n_tab - 1);
    const int t = full ? (e >> LOG_FULL) : e / (nqs * 32);
    const int n = e - t * (nqs * 32);
    xv[u] = *reinterpret_cast<const uint2*>(xs + int64_t(t) * a.C + 4 * n);
  }
  asm volatile("" ::: "memory");  // keep the activation loads ahead of the plane loads
  // plane i of quad q for row r at planes[(i nq + q) R + r]; parameters of
  // group column j at [(i gpr + j) R + r]; quad q lies in group q / qpg
  const int64_t R = a.R;
  const int64_t pstride = a.nq * R, astride = a.gpr * R;
  const int64_t rc = live ? r : R - 1;
  const u32x4* pp = reinterpret_cast<const u32x4*>(a.planes) + q0 * R + rc;
  const uint32_t qpg = uint32_t(a.qpg);
  const uint32_t j0 = uint32_t(q0) / qpg, rem0 = uint32_t(q0) - j0 * qpg;
  u32x4 pw[QPS][K];
  float al[QPS][K], zz[QPS];
#pragma unroll
  for (int qq = 0; qq < QPS; ++qq) {
    const int qc = min(qq, nqs - 1);
    const int64_t j = int64_t(j0 + (rem0 + uint32_t(qc)) / qpg);
    const uint16_t* ap = a.alpha16 + j * R + rc;
#pragma unroll
    for (int i = 0; i < K; ++i) {
      pw[qq][i] = pp[qc * R + i * pstride];
      al[qq][i] = f16_to_f32(ap[i * astride]);
    }
    zz[qq] = f16_to_f32(a.z16[j * R + rc]);
  }

  // table of nibble n: entry v is the sum of the activations of columns
  // 4 n + b with bit b of v set, in ascending bit order (built by doubling:
  // entries 2^b .. 2^(b+1) - 1 are entries 0 .. 2^b - 1 plus x_b)
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    // threads past the last table repeat it (identical values, same place)
    const int e = min(tid + 256 * u, n_tab - 1);
    {
      const int t = full ? (e >> LOG_FULL) : e / (nqs * 32);
      const int n = e - t * (nqs * 32);
      const float x0 = bf16_to_f32(uint16_t(xv[u].x)), x1 = bf16_to_f32(uint16_t(xv[u].x >> 16));
      const float x2 = bf16_to_f32(uint16_t(xv[u].y)), x3 = bf16_to_f32(uint16_t(xv[u].y >> 16));
      float L[16];
      L[0] = 0.0f;
      L[1] = x0;
      L[2] = x1;
      L[3] = x0 + x1;
#pragma unroll
      for (int v = 0; v < 4; ++v) L[4 + v] = L[v] + x2;
#pragma unroll
      for (int v = 0; v < 8; ++v) L[8 + v] = L[v] + x3;
      float4* dst = reinterpret_cast<float4*>(lut + t * PER_T + n * 16);
#pragma unroll
      for (int v = 0; v < 4; ++v) dst[v] = make_float4(L[4 * v], L[4 * v + 1], L[4 * v + 2], L[4 * v + 3]);
      // quad sum: the 32 nibble totals of a quad sit in 32 adjacent lanes
      // (tables are numbered quad-major and 256 u is a multiple of 32);
      // fixed xor-butterfly, written by the quad's first lane
      float tot = L[15];
#pragma unroll
      for (int msk = 16; msk >= 1; msk >>= 1) tot += __shfl_xor(tot, msk, 64);
      if ((tid & 31) == 0 && tid + 256 * u < n_tab) S[t * QPS + (n >> 5)] = tot;
    }
  }
  __syncthreads();
  if (!live) return;  // no barrier follows

  const char* lb = reinterpret_cast<const char*>(lut);
  float acc[T];
#pragma unroll
  for (int t = 0; t < T; ++t) acc[t] = 0.0f;
#pragma unroll
  for (int qq = 0; qq < QPS; ++qq) {
    if (qq >= nqs) break;
    float asum = 0.0f;
#pragma unroll
    for (int i = 0; i < K; ++i) asum += al[qq][i];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      float P[T];
#pragma unroll
      for (int t = 0; t < T; ++t) P[t] = 0.0f;
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        // byte offsets of the table entries: the even nibbles of the word
        // shifted to bits 8 n + 2 .. 8 n + 5, the odd ones likewise, so one
        // field extract gives 4 v for each nibble
        const uint32_t ev = (pw[qq][i][m] << 2) & 0x3C3C3C3Cu;
        const uint32_t od = (pw[qq][i][m] >> 2) & 0x3C3C3C3Cu;
        const uint32_t boff[8] = {byte_field<0>(ev), byte_field<0>(od), byte_field<8>(ev), byte_field<8>(od),
                                  byte_field<16>(ev), byte_field<16>(od), byte_field<24>(ev),
                                  byte_field<24>(od)};
#pragma unroll
        for (int nib = 0; nib < 8; ++nib) {
          const int row0 = ((qq * 32 + m * 8 + nib) * 16) * 4;  // byte offset of the nibble's table
#pragma unroll
          for (int t = 0; t < T; ++t)
            P[t] += *reinterpret_cast<const float*>(lb + boff[nib] + (row0 + t * PER_T * 4));
        }
      }
      const float a2 = 2.0f * al[qq][i];
#pragma unroll
      for (int t = 0; t < T; ++t) acc[t] += a2 * P[t];
    }
    const float zc = zz[qq] - asum;
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] += zc * S[t * QPS + qq];
  }
  float* out = a.out + int64_t(blockIdx.y) * T * a.R;
#pragma unroll
  for (int t = 0; t < T; ++t) out[int64_t(t) * a.R + r] = acc[t];
}

typedef __bf16 bf16x8b __attribute__((ext_vector_type(8)));
typedef float f32x4b __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_a8 __attribute__((aligned(8)));  // activations are 8-byte aligned

// The same product on MFMA (v_mfma_f32_16x16x32_bf16), for batches of four
// rows on and for small layers.  Per 128-column quad and plane the matrix cores
// sum the columns whose bit is set (tokens as M, 16 weight rows as N) and
// y += 2 alpha*_i P_i + (z* - sum_i alpha*_i) S as above.
//
// What bounds it is vector issue: every weight bit becomes a 16-bit operand.  A
// lane holds one 32-column word of a row and plane, and the columns of a
// fragment may come in any order that the activations share, so dword e of
// fragment s pairs columns b and b + 16, b = 15 - 4 s - e: with the word
// shifted left by 4 s - 1, their bits stand at 14 - e of the dword's two halves,
// and one v_and_b32 makes both bf16 values: 0, exactly, for a clear bit and a
// power of two for a set one, 2^1, 2^-63, 2^-95, 2^-111 for e = 0 .. 3.  The
// activations carry the rest (kUnit 2^-1, 2^63, ..): the products are kUnit x b,
// exactly, and one more product with constant columns gives kUnit S.  16
// instructions and four shifts per word and plane, where a 256-entry table in
// LDS was bound by its 16-byte reads.  (Bits expanded as (w & mask) | constant, the
// sign among them, took a shift less, 0.1 to 0.3 us in products of 3 to 8 us, but
// left a clear bit +-1/2, 2^-32 or 2^-64 of its activation.)
// An activation of 2^32 or more (or not finite) overflows its scaling, and what
// comes out not finite is added up again column by column (bcq_plain_sum).
//
// A wavefront takes 16 RT rows of its quads; the W wavefronts of a workgroup
// split the quads of the same rows and add up in LDS in a fixed order, so that
// most shapes need no partial rows and no second launch.  Each wavefront loads
// its quad's activations once, coalesced, pairs and scales them and reads the
// fragments back from its own LDS region (fragments loaded from memory touched
// 64 lines an instruction and were the bound: 58 us).  With RT = 2 a plane is
// one 8-byte load per lane, and v_permlane32_swap sorts words and parameters
// to the two row tiles.
// Measured (T = 8, g = 128; the table-expanded 32 x 32 x 16 form with partial rows
// before): 28672 x 8192, k = 3: 37 us against 45; 8192 x 28672: 34 against 45;
// 4096 x 4096, k = 4: 6.8 against 9.5 (one launch instead of two).  With the signed
// expansion 38, 35 and 6.7; its error against 64 bits was 1.3e-7, now 1.2e-7.
//
// One 128-column quad of 16 RT rows as a wavefront loads it: plane words,
// parameters (binary16) and this lane's 32 activations.
template <int K, int RT>
struct BcqQuad {
  uint32_t w[K][RT];
  uint16_t a[K], z;
  u32x4 x[2];
};

constexpr float kUnit = 0x1p-15f;

// Token tok's product with row r over quads q .. q_end - 1, one column at a time:
// the definition, for what overflows a fragment.  An infinite activation enters
// the sums of the bits that are set at its column and no others.
template <int K>
__device__ __forceinline__ float bcq_plain_sum(const BcqArgs& a, int tok, int64_t r, int64_t q, int64_t q_end) {
  float y = 0.0f;
#pragma unroll 1
  for (; q < q_end; ++q) {
    const int64_t j = q / a.qpg;
    float S = 0.0f, P[K] = {}, asum = 0.0f;
#pragma unroll 1
    for (int m = 0; m < 4; ++m) {
      uint32_t w[K];
#pragma unroll
      for (int i = 0; i < K; ++i) w[i] = a.planes[((i * a.nq + q) * a.R + r) * 4 + m];
#pragma unroll 1
      for (int c = 0; c < 32; ++c) {
        const float x = bf16_to_f32(a.X[tok * a.C + q * 128 + 32 * m + c]);
        S += x;
#pragma unroll
        for (int i = 0; i < K; ++i)
          if ((w[i] >> c) & 1u) P[i] += x;
      }
    }
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const float av = f16_to_f32(a.alpha16[(i * a.gpr + j) * a.R + r]);
      asum += av;
      y = __builtin_fmaf(2.0f * av, P[i], y);
    }
    y = __builtin_fmaf(f16_to_f32(a.z16[j * a.R + r]) - asum, S, y);
  }
  return y;
}

// Workgroup (bx, by): the 16 RT rows of row block rb0 + bx, quads qps by .. + qps - 1;
// wavefront w takes every W-th of them.
template <int K, int RT, int W>
__global__ __launch_bounds__(64 * W) void bcq_mfma_kernel(BcqArgs a, int T) {
  constexpr int ROWS = 16 * RT;
  constexpr int XLD = 17;  // 16-byte chunks per token (16 and one of padding: 8 tokens in distinct banks)
  __shared__ u32x4 xs[W][8 * XLD];
  __shared__ float red[W][8][ROWS];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, kg = lane >> 4;
  const int64_t R = a.R, r0 = (a.rb0 + blockIdx.x) * ROWS;
  // rows past R are loaded from the last one
  const uint32_t row = uint32_t(min(r0 + n + (RT == 2 ? 16 * (kg >> 1) : 0), R - 1) - r0);
  const int word = RT == 2 ? ((kg & 1) << 1) | (kg >> 1) : kg;  // of the quad's four, in the lane's fragments
  const int64_t q_end = min<int64_t>(a.nq, int64_t(blockIdx.y + 1) * a.qps);
  int64_t q = int64_t(blockIdx.y) * a.qps + wave;
  // 32-bit lane offsets from uniform bases (the quad and the wavefront are
  // uniform).  This lane loads columns 32 xw + 8 xc .. + 7 and the 8 sixteen
  // on, of token xt (tokens past T repeat the last, unused).
  const int xt = lane >> 3, xw = (lane >> 1) & 3, xc = lane & 1;
  const uint32_t xoff = 2u * (uint32_t(min(xt, T - 1)) * uint32_t(a.C) + 32u * xw + 8u * xc);
  u32x4* xput = &xs[wave][xt * XLD + 4 * xw + 2 * (1 - xc)];
  const u32x4* xget = &xs[wave][(n & 7) * XLD + 4 * word];
  const uint32_t woff = row * 16 + (RT == 2 ? 8 * (kg & 1) : 4 * kg), poff = row * 2;
  auto at = [](const void* base, uint32_t off) { return static_cast<const char*>(base) + off; };

  auto load = [&](BcqQuad<K, RT>& d, int64_t qq) {
    const int64_t j = a.qpg == 1 ? qq : int64_t((uint64_t(qq) * a.qpg_inv) >> 32);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const uint32_t* pp = a.planes + ((i * a.nq + qq) * R + r0) * 4;
      if constexpr (RT == 2) {
        const uint2 v = *reinterpret_cast<const uint2*>(at(pp, woff));
        d.w[i][0] = v.x;
        d.w[i][1] = v.y;
      } else {
        d.w[i][0] = *reinterpret_cast<const uint32_t*>(at(pp, woff));
      }
      d.a[i] = *reinterpret_cast<const uint16_t*>(at(a.alpha16 + (i * a.gpr + j) * R + r0, poff));
    }
    d.z = *reinterpret_cast<const uint16_t*>(at(a.z16 + j * R + r0, poff));
    const uint16_t* xq = a.X + qq * 128;
    d.x[0] = *reinterpret_cast<const u32x4_a8*>(at(xq, xoff));
    d.x[1] = *reinterpret_cast<const u32x4_a8*>(at(xq + 16, xoff));
  };

  constexpr uint32_t m[4] = {0x40004000u, 0x20002000u, 0x10001000u, 0x08000800u};
  const u32x4 sums = {m[0], m[1], m[2], m[3]};
  constexpr float scale[4] = {0.5f * kUnit, 0x1p63f * kUnit, 0x1p95f * kUnit, 0x1p111f * kUnit};
  f32x4b y[RT];
#pragma unroll
  for (int t = 0; t < RT; ++t) y[t] = f32x4b{0.0f, 0.0f, 0.0f, 0.0f};

  auto mul = [&](BcqQuad<K, RT>& d) {
    // chunk s, dword e: columns b and b + 16 of the word, b = 15 - 4 s - e.  (An odd
    // column's fp32 value keeps the even one's bits below it: they are cut off
    // again, and where the odd one is 0 they are worth less than 2^-133.)
    bf16x8b xa[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = (7 - 4 * h - e) >> 1;
        const uint32_t x0 = (e & 1) ? d.x[0][i] << 16 : d.x[0][i], x1 = (e & 1) ? d.x[1][i] << 16 : d.x[1][i];
        v[e] = __builtin_amdgcn_perm(__float_as_uint(__uint_as_float(x1) * scale[e]),
                                     __float_as_uint(__uint_as_float(x0) * scale[e]), 0x07060302u);
      }
      xput[h] = v;
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): written (read by this wavefront only)
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int s = 0; s < 4; ++s) xa[s] = __builtin_bit_cast(bf16x8b, xget[s]);
    f32x4b S = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < 4; ++s)
      S = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[s], __builtin_bit_cast(bf16x8b, sums), S, 0, 0, 0);
    uint32_t al[K][RT], zz[RT];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      al[i][0] = d.a[i];
      if constexpr (RT == 2) {
        const auto wv = __builtin_amdgcn_permlane32_swap(d.w[i][0], d.w[i][1], false, false);
        d.w[i][0] = wv[0];
        d.w[i][1] = wv[1];
        const auto av = __builtin_amdgcn_permlane32_swap(d.a[i], d.a[i], false, false);
        al[i][0] = av[0];
        al[i][1] = av[1];
      }
    }
    zz[0] = d.z;
    if constexpr (RT == 2) {
      const auto zv = __builtin_amdgcn_permlane32_swap(d.z, d.z, false, false);
      zz[0] = zv[0];
      zz[1] = zv[1];
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
      const float z = f16_to_f32(uint16_t(zz[t]));
      float asum = 0.0f;
#pragma unroll
      for (int i = 0; i < K; ++i) {
        const float av = f16_to_f32(uint16_t(al[i][t]));
        asum += av;
        f32x4b P = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const uint32_t w = s == 0 ? d.w[i][t] >> 1 : d.w[i][t] << (4 * s - 1);
          const u32x4 b = {w & m[0], w & m[1], w & m[2], w & m[3]};
          P = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[s], __builtin_bit_cast(bf16x8b, b), P, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) y[t][r] = __builtin_fmaf(2.0f * av, P[r], y[t][r]);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) y[t][r] = __builtin_fmaf(z - asum, S[r], y[t][r]);
    }
  };

  // The next quad's loads are in flight while one is multiplied; past the last
  // they repeat it, so that no branch surrounds them (behind one, the compiler
  // waits for every load in flight before each use).
  if (q < q_end) {
    BcqQuad<K, RT> d0, d1;
    load(d0, q);
    for (;;) {
      const int64_t q1 = q + W, q2 = q1 + W;
      load(d1, q1 < q_end ? q1 : q);
      __builtin_amdgcn_sched_barrier(0);
      mul(d0);
      if (q1 >= q_end) break;
      load(d0, q2 < q_end ? q2 : q1);
      __builtin_amdgcn_sched_barrier(0);
      mul(d1);
      if (q2 >= q_end) break;
      q = q2;
    }
  }

  if (kg < 2) {
#pragma unroll
    for (int t = 0; t < RT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][4 * kg + r][16 * t + n] = (1.0f / kUnit) * y[t][r];
  }
  __syncthreads();
  const int rr = threadIdx.x % ROWS;
#pragma unroll
  for (int tok = threadIdx.x / ROWS; tok < 8; tok += 64 * W / ROWS) {
    if (tok >= T || r0 + rr >= R) break;
    float s = 0.0f;
#pragma unroll
    for (int w = 0; w < W; ++w) s += red[w][tok][rr];
    if (!(fabsf(s) < INFINITY)) s = bcq_plain_sum<K>(a, tok, r0 + rr, int64_t(blockIdx.y) * a.qps, q_end);
    a.out[(int64_t(blockIdx.y) * T + tok) * R + r0 + rr] = s;
  }
}

// Y[t][r] = sum over slabs of the partial rows, slabs in ascending order.
__global__ __launch_bounds__(256) void bcq_reduce_kernel(const float* __restrict__ part, float* __restrict__ Y,
                                                         int64_t n, int slabs) {
  const int64_t idx = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= n) return;
  // up to 32 independent loads in flight (one memory round trip for most
  // shapes), added in slab order
  float s = 0.0f;
  for (int b0 = 0; b0 < slabs; b0 += 32) {
    float v[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) v[j] = b0 + j < slabs ? part[int64_t(b0 + j) * n + idx] : 0.0f;
#pragma unroll
    for (int j = 0; j < 32; ++j)
      if (b0 + j < slabs) s += v[j];
  }
  Y[idx] = s;
}

// Quads per slab of the table kernel, which sizes the workspace: the most (up to
// 4) that still give >= 512 workgroups.  The MFMA kernel needs at most a quarter
// of its slabs.
int bcq_quads_per_slab(int64_t R, int64_t C) {
  const int64_t rb = (R + 255) / 256, nq = C / 128;
  for (int qps = 4; qps > 1; qps >>= 1)
    if (rb * ((nq + qps - 1) / qps) >= 512) return qps;
  return 1;
}

int64_t bcq_slabs(int64_t R, int64_t C) {
  const int qps = bcq_quads_per_slab(R, C);
  return (C / 128 + qps - 1) / qps;
}

template <int K, int T, int QPS>
static void launch_mm(const BcqArgs& a, dim3 grid, hipStream_t st) {
  hipLaunchKernelGGL((bcq_matmul_kernel<K, T, QPS>), grid, dim3(256), 0, st, a);
}

template <int K, int T>
static void launch_mm_q(const BcqArgs& a, dim3 grid, hipStream_t st) {
  if (a.qps == 4) launch_mm<K, T, 4>(a, grid, st);
  else if (a.qps == 2) launch_mm<K, T, 2>(a, grid, st);
  else launch_mm<K, T, 1>(a, grid, st);
}

template <int K>
static void launch_mm_t(const BcqArgs& a, int T, dim3 grid, hipStream_t st) {
  switch (T) {
    case 1: launch_mm_q<K, 1>(a, grid, st); break;
    case 2: launch_mm_q<K, 2>(a, grid, st); break;
    default: launch_mm_q<K, 3>(a, grid, st); break;
  }
}

template <int K>
static void launch_mfma(const BcqArgs& a, int T, int rt, int w, dim3 grid, hipStream_t st) {
  if (rt == 1) hipLaunchKernelGGL((bcq_mfma_kernel<K, 1, 8>), grid, dim3(512), 0, st, a, T);
  else if (w == 1) hipLaunchKernelGGL((bcq_mfma_kernel<K, 2, 1>), grid, dim3(64), 0, st, a, T);
  else if (w == 8) hipLaunchKernelGGL((bcq_mfma_kernel<K, 2, 8>), grid, dim3(512), 0, st, a, T);
  else hipLaunchKernelGGL((bcq_mfma_kernel<K, 2, 16>), grid, dim3(1024), 0, st, a, T);
}

// Whether the table form takes the product; slabs and q: the MFMA form's column
// slabs and its quads a wavefront.  Never from four rows on, where the MFMA form's
// time does not grow with the batch.  Below:
//   above 21 M weights, where the tables read the bits at 4 TB/s (28672 x 8192, k = 3,
//   one row: 23.5 us against 36; 2000 x 12288, k = 4: 10.1 against 12.0);
//   one quad and many rows, where the tables need no second launch either (one row,
//   k = 3: 40000 x 128 3.6 us against 4.0, 28672 3.6 against 3.4; three rows: 65536 5.0 against
//   4.2, 128256 5.7 against 5.6);
//   one row of wide layers with three and four planes (28672 x 640, k = 3 6.6 us against
//   6.9, 24000 6.3 against 6.3);
//   rows whose chain of quads, at 0.5 to 1 us a quad, is longer than the tables' two
//   launches (one row, k = 4: 2048 x 7168 7.3 us against 9.2, 5120 7.2 against 7.4; two
//   rows 8.6 against 9.3, 6144 8.3 against 8.2), or that the MFMA form gives a second
//   launch of its own for two slabs (2048 x 8192, one row, k = 3: 7.2 against 8.2).
// Elsewhere the MFMA form's single launch counts (4096 x 4096, one row, k = 3: 6.3 us
// against 5.7; 512 x 28672: 12.9 against 9.7).
static bool table_takes(const BcqMatmulLaunch& p, int64_t nq, int64_t slabs, int q) {
  if (p.T > 3) return false;
  if (p.R * p.C > (int64_t(5) << 22)) return true;
  if (nq == 1) return p.R > 32768 * p.T;
  if (p.R >= 8192) return p.T == 1 && nq > 2 && p.k >= 3 && p.R >= (p.k == 4 && nq > 4 ? 20000 : 28672);
  return (slabs > 1 && p.T == 1 && p.k > 1 && nq < 96) || ((slabs == 1 || p.T == 1) && q + p.k >= 9 + p.T);
}

// Slabs for between one and two 32-row workgroups a CU: the CUs with two are twice as
// long as the others; S slabs cut that to ceil(rb S / 256) / S of a row block's time
// (0.04 k us a quad) for a second launch and its sums (3 + S us).  9000 x 28672, 4 rows,
// k = 4: 51 us against 79 (58 in the form before); 12000 x 16384 37 against 48.
static int64_t fill_slabs(int64_t rb, int64_t nq, int k) {
  int64_t best = 1;
  double t = 2.0 * 0.04 * double(k * nq);
  for (int64_t s = 2; s <= 4; ++s) {
    const double u = double((rb * s + 255) / 256) / double(s) * 0.04 * double(k * nq) + 3.0 + double(s);
    if (u < t) {
      t = u;
      best = s;
    }
  }
  return best;
}

hipError_t launch_bcq_matmul(const BcqMatmulLaunch& p, hipStream_t st) {
  BcqArgs a;
  a.rb0 = 0;
  a.X = p.X;
  a.planes = p.planes;
  a.alpha16 = p.alpha16;
  a.z16 = p.z16;
  a.R = p.R;
  a.C = p.C;
  a.nq = p.C / 128;
  a.gpr = p.C / p.g;
  a.qpg = p.g / 128;
  a.qpg_inv = a.qpg > 1 ? uint32_t(((uint64_t(1) << 32) + a.qpg - 1) / a.qpg) : 0;
  // The MFMA form: 16 rows a workgroup where that gives more workgroups than 32
  // would leave CUs busy; eight wavefronts over a row's quads, 16 where one
  // 32-row workgroup a CU and long rows leave eight alone (8192 x 28672, k = 3: 34 us
  // against 37; 9000 x 28672, more workgroups than CUs, 64 against 60), one where
  // there are one or two quads (128256 x 256, 4 rows, k = 3: 7.9 us against 16.5 with
  // idle ones).
  const int rt = p.R >= 8192 ? 2 : 1;
  const int64_t rb = (p.R + 16 * rt - 1) / (16 * rt);
  const int w = rt == 1 ? 8 : a.nq <= 2 && rb > 512 ? 1 : a.nq >= 128 && rb <= 256 ? 16 : 8;
  // Column slabs where the rows alone leave CUs idle and a wavefront would still
  // have four quads (512 x 28672: 9.7 us with 7 slabs, 23 with one): as many as fill
  // the CUs once, or three where that is one and three nearly fill them twice (4
  // rows, k = 3: 1536 x 28672 15.7 us against 17.0 with a slab more, 2560 x 16384 12.1
  // with three against 15.2 with two).
  int64_t slabs = rb <= 128   ? 256 / rb
                  : rb <= 170 ? (a.nq >= 96 ? 3 : 1)
                  : rb < 256  ? (a.nq >= 192 ? 2 : 1)
                  : rb > 256 && rb < 512 ? fill_slabs(rb, a.nq, p.k)
                              : 1;
  if (slabs > a.nq / (4 * w)) slabs = a.nq / (4 * w);
  if (slabs < 1) slabs = 1;
  const int64_t qps = (a.nq + slabs - 1) / slabs;
  slabs = (a.nq + qps - 1) / qps;
  if (!table_takes(p, a.nq, slabs, int((qps + w - 1) / w))) {
    a.qps = int(qps);
    a.out = slabs == 1 ? p.Y : p.partials;
    // a launch takes fewer than 2^32 threads
    constexpr int64_t kMaxBlocks = int64_t(1) << 21;
    for (a.rb0 = 0; a.rb0 < rb; a.rb0 += kMaxBlocks) {
      const dim3 grid{unsigned(rb - a.rb0 < kMaxBlocks ? rb - a.rb0 : kMaxBlocks), unsigned(slabs), 1u};
      switch (p.k) {
        case 1: launch_mfma<1>(a, p.T, rt, w, grid, st); break;
        case 2: launch_mfma<2>(a, p.T, rt, w, grid, st); break;
        case 3: launch_mfma<3>(a, p.T, rt, w, grid, st); break;
        default: launch_mfma<4>(a, p.T, rt, w, grid, st); break;
      }
    }
  } else {
    a.qps = bcq_quads_per_slab(p.R, p.C);
    slabs = (a.nq + a.qps - 1) / a.qps;
    a.out = slabs == 1 ? p.Y : p.partials;
    const dim3 grid(unsigned((p.R + 255) / 256), unsigned(slabs));
    switch (p.k) {
      case 1: launch_mm_t<1>(a, p.T, grid, st); break;
      case 2: launch_mm_t<2>(a, p.T, grid, st); break;
      case 3: launch_mm_t<3>(a, p.T, grid, st); break;
      default: launch_mm_t<4>(a, p.T, grid, st); break;
    }
  }
  if (slabs > 1) {
    const int64_t n = int64_t(p.T) * p.R;
    hipLaunchKernelGGL(bcq_reduce_kernel, dim3(unsigned((n + 255) / 256)), dim3(256), 0, st, p.partials, p.Y, n,
                       int(slabs));
  }
  return hipGetLastError();
}

}  // namespace uq
