// Head-wise rotation calibration (TurboESM Sec. 3.2): for the post-RoPE keys
// X (ncal x 64) of one head, Pi = V^T where X = U Sigma V^T.
//
// One block of 16 waves per head. The Gram matrix G = X^T X is accumulated in
// fp64 on the matrix cores and diagonalized in LDS by cyclic Jacobi rotations
// in the round-robin (tournament) order: each of the 63 rounds of a sweep
// applies 32 disjoint plane rotations at once. Eigenvalues of G are sigma^2;
// eigenvectors are the right singular vectors. Rows of Pi are ordered by
// descending sigma and signed so that each row's largest-magnitude entry is
// positive (lowest index on ties).
#include <algorithm>

#include "tq_device.hpp"
#include "tq_internal.hpp"

namespace tq {

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

constexpr int kMaxSweeps = 40;
constexpr int kRotWaves = 16;
constexpr int kRotThreads = kRotWaves * 64;
constexpr int kGramParts = 4;
constexpr int kGramBlocks = 10;   // 16 x 16 blocks (ib, jb), ib <= jb, of the symmetric G

struct RotSmem {
  double G[kDim * kDim];
  double V[kDim * kDim];
  double part[kGramParts][kGramBlocks * 256];
  double c[kPairs], s[kPairs];
  double off[kRotWaves], dia[kRotWaves];
  double sign[kDim];
  int rank[kDim];
};

// Pairs of a round: players 0 (fixed) and 1 .. 63 (turning). Pair k's members
// are positions k and 63 - k: over k both run through consecutive columns, so
// the 32 lanes of a half wave that read a row at them meet no bank twice.
__device__ __forceinline__ int tournament_player(int pos, int round) {
  const int p = pos - 1 + round;
  return pos == 0 ? 0 : (p >= kDim - 1 ? p - (kDim - 1) : p) + 1;
}

// What bounds it: the chain of about 9 sweeps x 63 rounds, each the rotations'
// angles (one wave) and then the update of G and V, 128 KB of LDS traffic on
// one compute unit. An update applies both sides of a 2 x 2 block of G in one
// thread (a block belongs to one pair of rotations, so no other thread reads
// it), where columns and rows one after the other cost a second pass and a
// third barrier. An angle's tangent needs no full precision (what it leaves
// of g_pq goes in the next sweep), so it is formed from the hardware's
// reciprocal and square root estimates; the rotation itself is orthogonal to
// fp64 rounding, as cos is refined to that and sin is tan times it.
// 20 heads x 4096 keys: 0.59 ms (0.5 ms of it the rounds), 5.23 ms with a wave
// per 16 columns of G from LDS and columns and rows turned one after the other.
__global__ __launch_bounds__(kRotThreads) void calibrate_kernel(const float* x, int ncal, float* pi_out,
                                                                float* sing_out) {
  __shared__ RotSmem sm;
  const int head = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const float* X = x + (int64_t)head * ncal * kDim;

  // ---- Gram matrix in fp64: a wave takes 4 vectors per step (lane group
  // lane / 16 one vector), whose 16-column pieces are both operands of the
  // blocks' products (v_mfma_f64_16x16x4f64: A[i][k] in lane i + 16 k,
  // B[k][j] in lane j + 16 k, D[4 r + lane / 16][lane % 16] in register r).
  {
    f64x4 acc[kGramBlocks];
#pragma unroll
    for (int e = 0; e < kGramBlocks; ++e) acc[e] = f64x4{0.0, 0.0, 0.0, 0.0};
    constexpr int kUnroll = 4;                 // steps whose loads are issued together
    for (int v0 = wave * 4; v0 < ncal; v0 += kRotWaves * 4 * kUnroll) {
      float xv[kUnroll][4];
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        const int v = v0 + u * kRotWaves * 4 + (lane >> 4);
        const float* row = X + (int64_t)min(v, ncal - 1) * kDim + (lane & 15);
#pragma unroll
        for (int ib = 0; ib < 4; ++ib) {
          const float w = row[16 * ib];
          xv[u][ib] = v < ncal ? w : 0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < kUnroll; ++u) {
        double xd[4];
#pragma unroll
        for (int ib = 0; ib < 4; ++ib) xd[ib] = (double)xv[u][ib];
        int e = 0;
#pragma unroll
        for (int ib = 0; ib < 4; ++ib)
#pragma unroll
          for (int jb = ib; jb < 4; ++jb, ++e)
            acc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(xd[ib], xd[jb], acc[e], 0, 0, 0);
      }
    }
    // the waves' sums, in a fixed order: four rounds into four partial matrices
    for (int rd = 0; rd < kRotWaves / kGramParts; ++rd) {
      if (wave / kGramParts == rd) {
        double* dst = sm.part[wave % kGramParts];
#pragma unroll
        for (int e = 0; e < kGramBlocks; ++e)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int at = e * 256 + (4 * r + (lane >> 4)) * 16 + (lane & 15);
            dst[at] = rd == 0 ? acc[e][r] : dst[at] + acc[e][r];
          }
      }
      __syncthreads();
    }
    for (int e = t; e < kDim * kDim; e += kRotThreads) {
      const int i = e >> 6, j = e & 63;
      const int lo = min(i, j), hi = max(i, j), ib = lo >> 4, jb = hi >> 4;
      // block (ib, jb) follows 4 + .. + (5 - ib) blocks; inside a diagonal block both halves hold the entry
      const int at = (ib * (9 - ib) / 2 + (jb - ib)) * 256 + (lo & 15) * 16 + (hi & 15);
      sm.G[e] = (sm.part[0][at] + sm.part[1][at]) + (sm.part[2][at] + sm.part[3][at]);
      sm.V[e] = i == j ? 1.0 : 0.0;
    }
  }
  __syncthreads();

  // ---- cyclic Jacobi, round-robin order
  for (int sweep = 0; sweep < kMaxSweeps; ++sweep) {
    // convergence: off-diagonal mass versus diagonal mass
    double off = 0.0, dia = 0.0;
#pragma unroll
    for (int e = t; e < kDim * kDim; e += kRotThreads) {
      const double g = sm.G[e];
      if ((e >> 6) == (e & 63)) dia += g * g; else off += g * g;
    }
    off = wave_sum_f64(off);
    dia = wave_sum_f64(dia);
    if (lane == 0) { sm.off[wave] = off; sm.dia[wave] = dia; }
    __syncthreads();
    double off_tot = 0.0, dia_tot = 0.0;
    for (int w = 0; w < kRotWaves; ++w) { off_tot += sm.off[w]; dia_tot += sm.dia[w]; }
    if (off_tot <= 1e-30 * dia_tot || off_tot == 0.0) break;

    for (int round = 0; round < kDim - 1; ++round) {
      const int k2 = t & 31, k1 = t >> 5;
      const int p2 = tournament_player(k2, round), q2 = tournament_player(kDim - 1 - k2, round);
      const int p1 = tournament_player(k1, round), q1 = tournament_player(kDim - 1 - k1, round);
      if (t < kPairs) {
        // tan = sign(h) d / (|h| + sqrt(h^2 + d^2)), h = g_qq - g_pp, d = 2 g_pq
        const double h = sm.G[q2 * kDim + q2] - sm.G[p2 * kDim + p2], d = 2.0 * sm.G[p2 * kDim + q2];
        const double hd = fma(h, h, d * d);
        double tn = 0.0;
        if (d != 0.0 && hd != 0.0) {
          const double den = fabs(h) + hd * __builtin_amdgcn_rsq(hd);
          tn = (h >= 0.0 ? d : -d) * __builtin_amdgcn_rcp(den);
        }
        const double w = fma(tn, tn, 1.0);
        double c = __builtin_amdgcn_rsq(w);
#pragma unroll
        for (int i = 0; i < 2; ++i) c = c * fma(-0.5 * w, c * c, 1.5);   // Newton's step for 1 / sqrt(w)
        sm.c[t] = c;
        sm.s[t] = tn * c;
      }
      __syncthreads();
      const double c1 = sm.c[k1], s1 = sm.s[k1], c2 = sm.c[k2], s2 = sm.s[k2];
      // G <- J^T G J on the block of rows p1, q1 and columns p2, q2
      const double gpp = sm.G[p1 * kDim + p2], gpq = sm.G[p1 * kDim + q2];
      const double gqp = sm.G[q1 * kDim + p2], gqq = sm.G[q1 * kDim + q2];
      const double v0p = sm.V[k1 * kDim + p2], v0q = sm.V[k1 * kDim + q2];
      const double v1p = sm.V[(k1 + 32) * kDim + p2], v1q = sm.V[(k1 + 32) * kDim + q2];
      const double app = c2 * gpp - s2 * gpq, apq = s2 * gpp + c2 * gpq;
      const double aqp = c2 * gqp - s2 * gqq, aqq = s2 * gqp + c2 * gqq;
      sm.G[p1 * kDim + p2] = c1 * app - s1 * aqp;
      sm.G[p1 * kDim + q2] = c1 * apq - s1 * aqq;
      sm.G[q1 * kDim + p2] = s1 * app + c1 * aqp;
      sm.G[q1 * kDim + q2] = s1 * apq + c1 * aqq;
      // V <- V J on columns p2, q2 of rows k1 and k1 + 32
      sm.V[k1 * kDim + p2] = c2 * v0p - s2 * v0q;
      sm.V[k1 * kDim + q2] = s2 * v0p + c2 * v0q;
      sm.V[(k1 + 32) * kDim + p2] = c2 * v1p - s2 * v1q;
      sm.V[(k1 + 32) * kDim + q2] = s2 * v1p + c2 * v1q;
      __syncthreads();
    }
  }

  // ---- order by descending eigenvalue, canonical signs, write Pi and sigma
  __syncthreads();
  if (t < kDim) {
    const double lt = sm.G[t * kDim + t];
    int rank = 0;
    for (int b = 0; b < kDim; ++b) {
      const double lb = sm.G[b * kDim + b];
      rank += (lb > lt || (lb == lt && b < t)) ? 1 : 0;
    }
    sm.rank[t] = rank;
    // column t of V is the eigenvector of eigenvalue lt
    int arg = 0;
    double best = -1.0;
    for (int k = 0; k < kDim; ++k) {
      const double v = fabs(sm.V[k * kDim + t]);
      if (v > best) { best = v; arg = k; }
    }
    sm.sign[t] = (sm.V[arg * kDim + t] < 0.0) ? -1.0 : 1.0;
    if (sing_out) sing_out[(int64_t)head * kDim + rank] = (float)sqrt(lt > 0.0 ? lt : 0.0);
  }
  __syncthreads();
  for (int e = t; e < kDim * kDim; e += kRotThreads) {
    const int k = e >> 6, col = e & 63;
    pi_out[((int64_t)head * kDim + sm.rank[col]) * kDim + k] = (float)(sm.sign[col] * sm.V[e]);
  }
}

hipError_t launch_calibrate(const float* x, int nheads, int ncal, float* pi_out, float* sing_out,
                            hipStream_t st) {
  hipLaunchKernelGGL(calibrate_kernel, dim3(nheads), dim3(kRotThreads), 0, st, x, ncal, pi_out, sing_out);
  return hipGetLastError();
}

// ------------------------------------------- normalized coordinates of a head
// Both kernels below walk the normalized coordinates u = 8 x^ / ||x^|| of a
// head's calibration vectors (x^ = Pi x in fp64, x^ = x without Pi; a zero
// vector gives zeros), one block of 8 waves per head, and recompute them each
// time they are needed: a head's 64 ncal doubles do not fit in LDS, and no
// workspace is passed. The rotation runs on the matrix cores in fp64
// (v_mfma_f64_16x16x4f64: full fp64 products and sums): a wave takes 16
// vectors, contracts k in the order that leaves each lane 16 consecutive
// elements to load (step s of lane group g = lane / 16 takes k = 16 g + s, on
// both operands), and holds its share of Pi, 64 doubles per lane, in registers
// for the whole call (calibrate_lut_kernel needs more than the 256 that two waves
// per SIMD leave, and spills 33). Every lane ends with 16 coordinates of vector
// lane % 16; the norm is a sum over them and the four lanes that hold the vector. A walk of
// 4096 vectors takes 0.18 ms (calibrate_ebar_kernel) to 0.23 ms, of which the
// matrix products are about 0.13 ms at the rate that a large fp64 product
// reaches per compute unit; one lane per coordinate with the rows of Pi read
// from LDS took 1.45 ms.
constexpr int kCalWaves = 8;
constexpr int kCalThreads = kCalWaves * 64;
constexpr int kWaveVectors = 16;
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // (x has no alignment of its own)

struct HeadRotation {
  double a[4][16];   // a[db][s] = Pi[16 db + lane % 16][16 (lane / 16) + s]
};

__device__ __forceinline__ void load_rotation(HeadRotation& R, const float* P, int lane) {
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
      const f32x4u w = *reinterpret_cast<const f32x4u*>(P + (16 * db + (lane & 15)) * kDim + 16 * (lane >> 4) + 4 * s4);
#pragma unroll
      for (int j = 0; j < 4; ++j) R.a[db][4 * s4 + j] = (double)w[j];
    }
}

struct VectorPart {
  f32x4u w[4];
};

__device__ __forceinline__ VectorPart load_vector_part(const float* X, int v, int ncal, int lane) {
  const f32x4u* src = reinterpret_cast<const f32x4u*>(X + (int64_t)min(v, ncal - 1) * kDim + 16 * (lane >> 4));
  VectorPart p;
#pragma unroll
  for (int j = 0; j < 4; ++j) p.w[j] = src[j];
  return p;
}

// Calls f(u[16], live) for every 16 coordinates of every vector (live: the
// lane's vector exists), the block's waves taking 16 vectors each in turn;
// with every > 1, of one group of 16 in `every`.
template <class F>
__device__ __forceinline__ void each_coordinate(const float* X, int ncal, bool rot, const HeadRotation& R, int wave, int lane,
                                                int every, F f) {
  const int64_t step = (int64_t)kCalWaves * kWaveVectors * every;
  const int n = lane & 15;
  int64_t v0 = (int64_t)wave * kWaveVectors * every;
  auto load = [&](int64_t v) { return load_vector_part(X, (int)min(v + n, (int64_t)ncal - 1), ncal, lane); };
  VectorPart next = load(v0);
  for (; v0 < ncal; v0 += step) {
    double xh[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) xh[k] = (double)next.w[k >> 2][k & 3];
    next = load(v0 + step);
    if (rot) {
      f64x4 acc[4];
#pragma unroll
      for (int db = 0; db < 4; ++db) acc[db] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 16; ++s)
#pragma unroll
        for (int db = 0; db < 4; ++db)
          acc[db] = __builtin_amdgcn_mfma_f64_16x16x4f64(R.a[db][s], xh[s], acc[db], 0, 0, 0);
#pragma unroll
      for (int k = 0; k < 16; ++k) xh[k] = acc[k >> 2][k & 3];
    }
    double n2 = 0.0;
#pragma unroll
    for (int k = 0; k < 16; ++k) n2 = fma(xh[k], xh[k], n2);
    n2 += __shfl_xor(n2, 16, 64);
    n2 += __shfl_xor(n2, 32, 64);
    const double inv = 8.0 / sqrt(n2);
#pragma unroll
    for (int k = 0; k < 16; ++k) xh[k] = (n2 > 0.0) ? xh[k] * inv : 0.0;
    f(xh, v0 + n < ncal);
  }
}

// ------------------------------------------------------- table calibration
// Calibrated 8-level table per head (Sec. 3.3: calibrated, separate K and V
// tables): the 1-D Lloyd iteration (k-means) on every normalized coordinate.
// Per iteration: assign each u to the level whose midpoint interval holds it
// (u > t_m strictly counts, so a tie goes to the lower level), replace each
// level by the mean of its cell (an empty cell keeps its level), take the
// largest level change, sort, and stop once that change is below tol, or
// after max_iter iterations.
//
// An iteration needs, for its 7 midpoints t, only the count and the sum of
// the coordinates above t. A short walk over a sample of the vectors sizes
// kBins bins over [-8, 8] to hold about equally many coordinates; a full walk
// fills them with exact counts and sums, turned into prefix sums. A midpoint
// then needs the coordinates of its own bin one by one, and a third kind of
// walk collects those: around each midpoint a window of bins, as wide as
// kWindow coordinates allow and wider on the side the midpoint is moving to,
// whose coordinates are kept in LDS as fp64. Iterations then read LDS only,
// until a midpoint leaves its window and the next walk collects new ones: 100
// iterations over 4096 vectors take 3 to 6 such walks on random rotations
// and about 18 on an SVD basis, whose levels move further. A bin too full
// for a window (many equal coordinates) makes that iteration's walk count
// directly. Every decision compares the fp64 coordinate with the fp64
// midpoint, as a plain iteration over all coordinates does.
//
// Sums are kept as integers in units of 2^-sum_bits, so they do not depend on
// the order in which the lanes arrive. A vector's coordinates have mean square
// 1, so n of them sum to at most n in magnitude, and sum_bits = 62 - log2 n
// (44 at 4096 vectors, 36 at 2^20) cannot overflow. A coordinate is rounded by
// up to 2^-(sum_bits + 1), at most fp32's rounding of a level of at least
// 2^(24 - sum_bits). Where a level ends below that and coordinates below it
// exist, the table is made again by plain iterations with fp64 sums
// (plain_lloyd), so that levels far below the others keep their precision and
// stay apart.
//
// What bounds it: the walks, on the one compute unit that a head gets. 20
// heads x 4096 keys and random rotations take 1.73 ms (144 ms with a walk per
// iteration by one lane per coordinate); on the keys' SVD bases 8.6 ms, and
// unrotated keys 3.6 ms (37 ms and 37 ms with bins of equal width, whose
// middle ones overflow the windows there).
struct Mass {            // of a set of coordinates
  int64_t n, sum;
};

constexpr int kCoarse = 256;             // equal cells over [-8, 8], each of 2^j bins
constexpr int kCoarseBits = 11;          // (at most 2^11)
constexpr int kBins = 4096;
constexpr int kBinShare = 1900;          // 2 * 1900 + 256 <= kBins: sizes are rounded up to powers of two
constexpr int kWindow = 1536;
constexpr double kFixMagic = 6755399441055744.0;   // 1.5 * 2^52: adding it leaves an integer in the low bits

struct LutSmem {
  Mass below[kBins + 1];                 // mass of the bins below b
  union {
    double list[7][kWindow];             // the windows' coordinates
    uint32_t coarse[kCoarse];            // the sample's counts
  };
  uint8_t owner[kBins];                  // the window that holds a bin, 0xFF: none
  uint16_t cell[kCoarse];                // first bin * 16 + shift of a coarse cell
  int wa[7], wb[7], win[7];              // midpoint m: its window [wa, wb) and that window's list
  int listed[7];
  Mass above[2][7];
  Mass part[kCalWaves][8];               // a direct walk: each wave's cells
  Mass carry[kCalWaves];
  double plain[kCalWaves][8];            // plain iterations: each wave's cells
  int64_t plain_n[kCalWaves][8];
  int over, nan, tiny;
};

// Position of u on a grid of kCoarse << kCoarseBits steps over [-8, 8] (0 for NaN).
// (a walk's coordinates are within rounding of it; midpoints can lie outside).
__device__ __forceinline__ int grid_of(double u) {
  constexpr int kSteps = kCoarse << kCoarseBits;
  return min((int)fmin(fmax(fma(u, kSteps / 16.0, kSteps / 2.0), 0.0), (double)kSteps), kSteps - 1);
}

__device__ __forceinline__ int bin_of(const LutSmem& sm, double u) {
  const int g = grid_of(u);
  const int cell = sm.cell[g >> kCoarseBits];
  return (cell >> 4) + ((g & ((1 << kCoarseBits) - 1)) >> (cell & 15));
}

// u in units of 2^-sum_bits (unit = 2^sum_bits), to nearest.
__device__ __forceinline__ int64_t fixed_of(double u, double unit) {
  return __double_as_longlong(fma(u, unit, kFixMagic)) - __double_as_longlong(kFixMagic);
}

__device__ __forceinline__ void add_i64(int64_t& to, int64_t v) {
  atomicAdd(reinterpret_cast<unsigned long long*>(&to), (unsigned long long)v);
}

__device__ __forceinline__ int64_t wave_sum_i64(int64_t v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor((long long)v, o, 64);
  return v;
}

// Inclusive sum over the wave's lanes up to this one.
__device__ __forceinline__ int64_t wave_scan_i64(int64_t v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t w = __shfl_up((long long)v, o, 64);
    v += lane >= o ? w : 0;
  }
  return v;
}

// Levels in lanes k, k + 8, .. in ascending order (a NaN level, only ever the
// first, stays first).
__device__ __forceinline__ double ascending(double fresh, int k) {
  int rank = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const double lj = __shfl(fresh, j, 64);
    rank += (lj < fresh || ((lj == fresh || lj != lj) && j < k)) ? 1 : 0;
  }
  double lev = fresh;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const double lj = __shfl(fresh, j, 64);
    lev = __shfl(rank, j, 64) == k ? lj : lev;
  }
  return lev;
}

// The iteration as it is defined: a walk each, every lane summing its
// coordinates' cells in fp64 in a fixed order. (Not inlined: its registers
// would be spilled from calibrate_lut_kernel's loops.)
__device__ __attribute__((noinline)) double plain_lloyd(LutSmem& sm, const float* X, int ncal, const float* pi,
                                                        LutInit init, int max_iter, double tol) {
  const int lane = threadIdx.x & 63, k = lane & 7;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  HeadRotation R;
  if (pi) load_rotation(R, pi, lane);
  double lev = 0.0;
#pragma unroll
  for (int j = 0; j < 8; ++j) lev = k == j ? (double)init.c[j] : lev;
  for (int it = 0; it < max_iter; ++it) {
    double tm[7], sum[8];
    int n[8];
#pragma unroll
    for (int m = 0; m < 7; ++m) tm[m] = 0.5 * (__shfl(lev, m, 64) + __shfl(lev, m + 1, 64));
#pragma unroll
    for (int c = 0; c < 8; ++c) { sum[c] = 0.0; n[c] = 0; }
    each_coordinate(X, ncal, pi != nullptr, R, wave, lane, 1, [&](const double (&u)[16], bool live) {
      if (!live) return;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        int at = 0;
#pragma unroll
        for (int m = 0; m < 7; ++m) at += (u[j] > tm[m]) ? 1 : 0;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          sum[c] += at == c ? u[j] : 0.0;
          n[c] += at == c ? 1 : 0;
        }
      }
    });
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const double s = wave_sum_f64(sum[c]);
      const int64_t cnt = wave_sum_i64(n[c]);
      if (lane == 0) { sm.plain[wave][c] = s; sm.plain_n[wave][c] = cnt; }
    }
    __syncthreads();
    double s = 0.0;
    int64_t cnt = 0;
    for (int w = 0; w < kCalWaves; ++w) { s += sm.plain[w][k]; cnt += sm.plain_n[w][k]; }
    __syncthreads();
    const double fresh = cnt > 0 ? s / (double)cnt : lev;
    double delta = fabs(fresh - lev);
    delta = (delta == delta) ? delta : 0.0;
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) delta = fmax(delta, __shfl_xor(delta, o, 64));
    lev = ascending(fresh, k);
    if (delta < tol) break;                // (the same in every wave)
  }
  return lev;
}

__global__ __launch_bounds__(kCalThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void calibrate_lut_kernel(const float* x, int ncal, const float* pi, LutInit init, int max_iter, double tol,
                          int sum_bits, float* lut_out) {
  __shared__ LutSmem sm;
  const int head = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const float* X = x + (int64_t)head * ncal * kDim;
  const bool rot = pi != nullptr;
  const double unit = ldexp(1.0, sum_bits), least = ldexp(1.0, 24 - sum_bits);
  HeadRotation R;
  if (rot) load_rotation(R, pi + (int64_t)head * kDim * kDim, lane);
  if (t < 7) { sm.wa[t] = 0; sm.wb[t] = 0; }
  if (t == 0) { sm.over = 0; sm.nan = 0; sm.tiny = 0; }
  for (int c = t; c < kCoarse; c += kCalThreads) sm.coarse[c] = 0u;
  __syncthreads();

  // ---- a sample of about 512 vectors sizes the bins
  each_coordinate(X, ncal, rot, R, wave, lane, max(1, ncal >> 9), [&](const double (&u)[16], bool live) {
    if (!live) return;
#pragma unroll
    for (int k = 0; k < 16; ++k) atomicAdd(&sm.coarse[grid_of(u[k]) >> kCoarseBits], 1u);
  });
  __syncthreads();
  if (wave == 0) {
    // cell c gets 2^j >= kBinShare * (its share of the sample) bins, 1 <= 2^j <= 2^kCoarseBits
    uint32_t cnt[4];
    int64_t all = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) { cnt[j] = sm.coarse[lane * 4 + j]; all += cnt[j]; }
    all = wave_sum_i64(all);
    int bits[4], bins = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t want = (int64_t)cnt[j] * kBinShare;
      bits[j] = 0;
      while (bits[j] < kCoarseBits && (all << bits[j]) < want) ++bits[j];
      bins += 1 << bits[j];
    }
    int first = (int)wave_scan_i64(bins, lane) - bins;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      sm.cell[lane * 4 + j] = (uint16_t)(first * 16 + (kCoarseBits - bits[j]));
      first += 1 << bits[j];
    }
  }
  __syncthreads();
  for (int b = t; b < kBins; b += kCalThreads) sm.below[b] = Mass{0, 0};
  __syncthreads();

  // ---- histogram. A NaN coordinate (infinite inputs) belongs to cell 0, as
  // no comparison holds, and makes that cell's sum NaN.
  each_coordinate(X, ncal, rot, R, wave, lane, 1, [&](const double (&u)[16], bool live) {
    if (!live) return;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      if (u[k] != u[k]) {
        sm.nan = 1;
      } else {
        const int b = bin_of(sm, u[k]);
        add_i64(sm.below[b].n, 1);
        add_i64(sm.below[b].sum, fixed_of(u[k], unit));
        if (fabs(u[k]) < least && u[k] != 0.0) sm.tiny = 1;
      }
    }
  });
  __syncthreads();
  {
    // prefix sums of the bins: kPer bins per thread, then the waves in order
    constexpr int kPer = kBins / kCalThreads;
    Mass own[kPer], all{0, 0};
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      own[j] = all;
      all.n += sm.below[t * kPer + j].n;
      all.sum += sm.below[t * kPer + j].sum;
    }
    const Mass scan{wave_scan_i64(all.n, lane), wave_scan_i64(all.sum, lane)};
    if (lane == 63) sm.carry[wave] = scan;
    __syncthreads();
    Mass base{scan.n - all.n, scan.sum - all.sum};
    for (int w = 0; w < wave; ++w) { base.n += sm.carry[w].n; base.sum += sm.carry[w].sum; }
#pragma unroll
    for (int j = 0; j < kPer; ++j) sm.below[t * kPer + j] = Mass{base.n + own[j].n, base.sum + own[j].sum};
    if (t == kCalThreads - 1) sm.below[kBins] = Mass{base.n + all.n, base.sum + all.sum};
  }
  __syncthreads();

  // ---- iterations. Every wave keeps the levels (lane k, k + 8, ..: level k)
  // and computes them itself, so that one barrier per iteration is enough;
  // wave m < 7 looks after midpoint m.
  const int k = lane & 7;
  double lev = 0.0;
#pragma unroll
  for (int j = 0; j < 8; ++j) lev = k == j ? (double)init.c[j] : lev;
  const Mass total = sm.below[kBins];
  const bool any_nan = sm.nan != 0;
  double told = 0.0;                       // the wave's midpoint in the iteration before
  for (int it = 0; it < max_iter; ++it) {
    // midpoint k in lanes k, k + 8, .. (k < 7); one of a NaN level counts nothing
    const double mid = 0.5 * (lev + __shfl(lev, (lane + 1) & 7, 64));
    const bool on = k < 7 && mid == mid;
    const double th = __shfl(mid, min(wave, 6), 64);
    const int bin = bin_of(sm, mid);
    const bool out = on && !(bin >= sm.wa[min(k, 6)] && bin < sm.wb[min(k, 6)]);
    bool direct = false;
    if (__builtin_amdgcn_ballot_w64(out) != 0) {     // (the same in every wave)
      __syncthreads();                               // (every wave has read the windows)
      if (wave < 7 && th == th) {
        // the widest window around bin bt: all of that bin, and on each side
        // the bins that the rest of the list has room for, 7/8 of it ahead
        const int bt = bin_of(sm, th);
        const int64_t lo = sm.below[bt].n, hi = sm.below[bt + 1].n, rest = kWindow - (hi - lo);
        const double move = it == 0 ? 0.0 : th - told;
        const int64_t up = move > 0.0 ? rest - rest / 8 : (move < 0.0 ? rest / 8 : rest / 2), down = rest - up;
        if (rest < 0) {
          if (lane == 0) sm.over = 1;
        } else {
          int a0 = 0, a1 = bt;                       // smallest a with n[bt] - n[a] <= down
          while (a0 < a1) {
            const int half = (a0 + a1) >> 1;
            if (lo - sm.below[half].n <= down) a1 = half; else a0 = half + 1;
          }
          int b0 = bt + 1, b1 = kBins;               // largest b with n[b] - n[bt + 1] <= up
          while (b0 < b1) {
            const int half = (b0 + b1 + 1) >> 1;
            if (sm.below[half].n - hi <= up) b0 = half; else b1 = half - 1;
          }
          if (lane == 0) { sm.wa[wave] = a0; sm.wb[wave] = b0; }
        }
      }
      __syncthreads();
      direct = sm.over != 0;
      __syncthreads();
      if (wave == 0) {
        // windows do not overlap: midpoints are ascending, so a window starts
        // at the end of the one before, or is that one where it holds the midpoint
        int end = 0, last = 0;
        for (int m = 0; m < 7; ++m) {
          const double tm = __shfl(mid, m, 64);
          const int bm = bin_of(sm, tm);
          if (lane != 0) continue;
          if (direct || tm != tm) {                  // (a direct walk leaves no window)
            sm.wa[m] = 0;
            sm.wb[m] = 0;
            continue;
          }
          if (end > 0 && bm < end) {
            sm.wa[m] = sm.wa[last];
            sm.wb[m] = end;
            sm.win[m] = sm.win[last];
          } else {
            sm.wa[m] = max(sm.wa[m], end);
            end = sm.wb[m];
            sm.win[m] = m;
          }
          last = m;
        }
        if (lane == 0) sm.over = 0;
        if (lane < 7) sm.listed[lane] = 0;
      }
      __syncthreads();
      if (!direct) {
        for (int b = t; b < kBins; b += kCalThreads) {
          int w = 0xFF;
#pragma unroll
          for (int m = 0; m < 7; ++m) w = (b >= sm.wa[m] && b < sm.wb[m]) ? sm.win[m] : w;
          sm.owner[b] = (uint8_t)w;
        }
        __syncthreads();
        each_coordinate(X, ncal, rot, R, wave, lane, 1, [&](const double (&u)[16], bool live) {
          if (!live) return;
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int w = sm.owner[bin_of(sm, u[j])];
            if (u[j] == u[j] && w != 0xFF) {
              const int at = atomicAdd(&sm.listed[w], 1);
              if (at < kWindow) sm.list[w][at] = u[j];   // (the window's count is at most kWindow)
            }
          }
        });
      } else {
        double tm[7];
#pragma unroll
        for (int m = 0; m < 7; ++m) tm[m] = __shfl(mid, m, 64);
        if (lane < 8) sm.part[wave][lane] = Mass{0, 0};
        each_coordinate(X, ncal, rot, R, wave, lane, 1, [&](const double (&u)[16], bool live) {
          if (!live) return;
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            int c = 0;
#pragma unroll
            for (int m = 0; m < 7; ++m) c += (u[j] > tm[m]) ? 1 : 0;
            if (u[j] == u[j]) {
              add_i64(sm.part[wave][c].n, 1);
              add_i64(sm.part[wave][c].sum, fixed_of(u[j], unit));
            }
          }
        });
      }
      __syncthreads();
    }

    // ---- the mass above the wave's midpoint
    Mass* const above = sm.above[it & 1];
    if (wave < 7 && th == th) {
      Mass s{0, 0};
      if (direct) {
        // the cells above the midpoint, counting the midpoints that are not NaN
        const int first = __popcll(__builtin_amdgcn_ballot_w64(lane <= wave && mid == mid));
        for (int w = 0; w < kCalWaves; ++w)
          for (int j = first; j < 8; ++j) { s.n += sm.part[w][j].n; s.sum += sm.part[w][j].sum; }
      } else {
        const int w = sm.win[wave], cnt = min(sm.listed[w], kWindow);
        for (int i = lane; i < cnt; i += 64) {
          const double u = sm.list[w][i];
          if (u > th) { s.n += 1; s.sum += fixed_of(u, unit); }
        }
        const Mass end = sm.below[sm.wb[wave]];
        s.n = wave_sum_i64(s.n) + (total.n - end.n);
        s.sum = wave_sum_i64(s.sum) + (total.sum - end.sum);
      }
      if (lane == 0) above[wave] = s;
    }
    told = th;
    __syncthreads();

    // ---- new levels: cell k holds the coordinates above exactly k midpoints
    Mass hi = total, lo{0, 0};             // above the cell's lower and upper midpoint
    int seen = 0;
#pragma unroll
    for (int m = 0; m < 7; ++m) {
      const double tm = __shfl(mid, m, 64);
      if (tm == tm) {
        ++seen;
        if (seen == k) hi = above[m];
        if (seen == k + 1) lo = above[m];
      }
    }
    const int64_t n = k <= seen ? hi.n - lo.n : 0;   // (fewer cells where a midpoint is NaN)
    double fresh = n > 0 ? ldexp((double)(hi.sum - lo.sum), -sum_bits) / (double)n : lev;
    if (k == 0 && any_nan) fresh = __longlong_as_double(0x7FF8000000000000ll);
    double delta = fabs(fresh - lev);
    delta = (delta == delta) ? delta : 0.0;
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) delta = fmax(delta, __shfl_xor(delta, o, 64));
    lev = ascending(fresh, k);
    if (delta < tol) break;                // (the same in every wave)
  }
  if (sm.tiny != 0 && __builtin_amdgcn_ballot_w64(fabs(lev) < ldexp(1.0, 24 - sum_bits)) != 0)
    lev = plain_lloyd(sm, X, ncal, pi ? pi + (int64_t)head * kDim * kDim : nullptr, init, max_iter, tol);
  if (t < 8) lut_out[(int64_t)head * 8 + t] = (float)lev;
}

hipError_t launch_calibrate_lut(const float* x, int nheads, int ncal, const float* pi, const float* init,
                                int max_iter, double tol, float* lut_out, hipStream_t st) {
  LutInit in;
  for (int m = 0; m < 8; ++m) in.c[m] = init[m];
  int log2n = 6;
  while (((int64_t)1 << log2n) < (int64_t)ncal * kDim) ++log2n;
  const int sum_bits = std::min(47, 62 - log2n);   // (47: a coordinate, at most 8, in fixed_of's 51 bits)
  hipLaunchKernelGGL(calibrate_lut_kernel, dim3(nheads), dim3(kCalThreads), 0, st, x, ncal, pi, in, max_iter, tol,
                     sum_bits, lut_out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- ebar
// Per-head mean absolute residual of the per-element correction (Sec. 3.4,
// Eq. 7): over every normalized coordinate of the head's calibration vectors,
// the mean of |u - c[idx]| with idx = #{m : u > (c_m + c_{m+1})/2} (fp64
// midpoints of the fp32 levels). Each lane sums its coordinates in fp64 in a
// fixed order, and the lanes' sums are added in a fixed order. A head whose
// table is not strictly ascending gets NaN. One walk: 0.18 ms at 4096 vectors
// (1.56 ms with one lane per coordinate).
__global__ __launch_bounds__(kCalThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void calibrate_ebar_kernel(const float* x, int ncal, const float* pi, const float* lut, float* ebar_out,
                           int stride) {
  __shared__ double s_sum[kCalWaves];
  const int head = blockIdx.x;
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const bool rot = pi != nullptr;
  HeadRotation R;
  if (rot) load_rotation(R, pi + (int64_t)head * kDim * kDim, lane);
  double c[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) c[m] = (double)lut[(int64_t)head * 8 + m];
  bool asc = true;
#pragma unroll
  for (int m = 0; m < 7; ++m) asc = asc && (c[m] < c[m + 1]);
  double th[7];
#pragma unroll
  for (int m = 0; m < 7; ++m) th[m] = 0.5 * (c[m] + c[m + 1]);
  double acc = 0.0;
  each_coordinate(x + (int64_t)head * ncal * kDim, ncal, rot, R, wave, lane, 1, [&](const double (&u)[16], bool live) {
    if (!live) return;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      double lv = c[0];
#pragma unroll
      for (int m = 0; m < 7; ++m) lv = (u[k] > th[m]) ? c[m + 1] : lv;
      acc += fabs(u[k] - lv);
    }
  });
  acc = wave_sum_f64(acc);
  if (lane == 0) s_sum[wave] = acc;
  __syncthreads();
  if (t == 0) {
    double total = 0.0;
    for (int w = 0; w < kCalWaves; ++w) total += s_sum[w];
    const double mean = total / ((double)ncal * kDim);
    ebar_out[(int64_t)head * stride] = asc ? (float)mean : __int_as_float(0x7FC00000);
  }
}

hipError_t launch_calibrate_ebar(const float* x, int nheads, int ncal, const float* pi, const float* lut,
                                 float* ebar_out, int stride, hipStream_t st) {
  hipLaunchKernelGGL(calibrate_ebar_kernel, dim3(nheads), dim3(kCalThreads), 0, st, x, ncal, pi, lut, ebar_out,
                     stride);
  return hipGetLastError();
}

}  // namespace tq
