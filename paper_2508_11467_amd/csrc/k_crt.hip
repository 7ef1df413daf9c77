// Split-precision FP64 products on the int8 matrix cores through the Chinese
// remainder theorem (the integer-modular emulation of Ozaki, Uchino and
// Imamura, "Ozaki Scheme II", 2025), for the vector-update products of eq.
// bdc-Mv2Bv-u-vt:
//
//   1. every row r of the left operand and every column of the right one is
//      scaled by a power of two 2^E_r so that its largest entry lies below
//      2^beta, and rounded to an integer (A', B');
//   2. for each of L pairwise coprime odd moduli m_l <= 255 the residues
//      A' mod m_l and B' mod m_l are taken in the balanced range
//      [-(m_l-1)/2, (m_l-1)/2] (they fit int8);
//   3. the residue matrices are multiplied on v_mfma_i32_16x16x64_i8 with
//      exact int32 accumulation, and each sum is reduced mod m_l again;
//   4. the integer A'B' is rebuilt from its L residues by the theorem's sum:
//      with y_l the inverse of M/m_l mod m_l (M = prod m_l) and v_l = A'B' y_l
//      mod m_l, A'B' = sum_l v_l (M/m_l) mod M, exact in integers (the factor
//      y_l is part of B's residues), then scaled back by 2^-(E_r + E_c) with a
//      single rounding to FP64.
//
// beta is chosen so that K 2^(2 beta) <= (M - 1)/2, M = prod m_l, hence
// |A'B'| lies inside the balanced range and step 4 recovers it exactly; it is
// capped at 55 so that |A'| <= 2^55 fits the seven bytes step 2 splits it into.  The
// only roundings are those of A and B to integers (at most half a unit of
// 2^-beta times the row's / column's largest entry) and the final conversion
// to FP64.  Residue planes are int8, k contiguous, rows padded to kCrtRowPad
// and k to kCrtKStep with zeros.
#include <algorithm>
#include <cmath>

#include "bdc_internal.h"
#include "crt.h"
#include "gemm128.h"

namespace bdc {
namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned int CrtWords __attribute__((ext_vector_type(4), aligned(4)));  // 16 bytes at any word

// ------------------------------------------------------------ moduli tables
// moduli in descending order; every table is computed at compile time
constexpr int kMod[kCrtMaxMod] = {255, 253, 251, 247, 241, 239, 233, 229,
                                  227, 223, 217, 211, 199, 197, 193, 191};

constexpr int mod_pos(long long a, int m) {
  const long long r = a % m;
  return (int)(r < 0 ? r + m : r);
}
constexpr int mod_inv(int a, int m) {
  // extended Euclid on (a mod m, m)
  long long r0 = m, r1 = mod_pos(a, m), t0 = 0, t1 = 1;
  while (r1 != 0) {
    const long long q = r0 / r1;
    const long long r2 = r0 - q * r1, t2 = t0 - q * t1;
    r0 = r1;
    r1 = r2;
    t0 = t1;
    t1 = t2;
  }
  return mod_pos(t0, m);
}
constexpr int balanced(int r, int m) { return r > (m - 1) / 2 ? r - m : r; }

typedef unsigned __int128 u128;
constexpr int kDigits = 15;  // signed base-256 digits of M/m_l < 2^118 (16 moduli)

template <int L>
struct CrtTables {
  unsigned pw[2][L][2];        // [right operand][l]: the bytes 2^(8 b) mod m_l (times y_l), b = 0..6
  unsigned dig[kDigits][4];    // [b]: digit b of M/m_l as the bytes l = 0..15
  int mlimb[4];                // M in signed 32-bit digits
  float part[8];               // 2^(16 k) / M
  unsigned long long mlo, hlo;
  long long mhi, hhi;          // M and (M - 1) / 2
};
template <int L>
constexpr CrtTables<L> make_tables() {
  CrtTables<L> t{};
  u128 M = 1;
  for (int l = 0; l < L; ++l) M *= (u128)kMod[l];
  for (int l = 0; l < L; ++l) {
    const int m = kMod[l];
    u128 c = M / (u128)m;
    const int y = mod_inv((int)(c % (u128)m), m);
    int p = 1;
    for (int b = 0; b < 7; ++b) {
      t.pw[0][l][b / 4] |= (unsigned)p << (8 * (b % 4));
      t.pw[1][l][b / 4] |= (unsigned)((p * y) % m) << (8 * (b % 4));
      p = (p * 256) % m;
    }
    for (int b = 0; b < kDigits; ++b) {
      const int r = (int)(c & 255), d = r > 127 ? r - 256 : r;
      t.dig[b][l / 4] |= ((unsigned)d & 255u) << (8 * (l % 4));
      c = (c >> 8) + (d < 0 ? 1 : 0);
    }
  }
  u128 c = M;
  for (int j = 0; j < 4; ++j) {
    t.mlimb[j] = (int)(unsigned)c;
    c = (c >> 32) + (t.mlimb[j] < 0 ? 1 : 0);
  }
  const double inv_m = 1.0 / ((double)(unsigned long long)(M >> 64) * 0x1p64 + (double)(unsigned long long)M);
  double p = 1.0;
  for (int k = 0; k < 8; ++k, p *= 65536.0) t.part[k] = (float)(p * inv_m);
  t.mlo = (unsigned long long)M;
  t.mhi = (long long)(M >> 64);
  t.hlo = (unsigned long long)((M - 1) / 2);
  t.hhi = (long long)((M - 1) / 2 >> 64);
  return t;
}
template <int L>
constexpr CrtTables<L> kTab = make_tables<L>();

// x (an integer-valued float, |x| < 2^24) mod m in the balanced range.  For
// odd m, x/m is never within 1/(2m) of a half-integer, so the rounded
// quotient is exact despite the rounding of x * (1/m), and the remainder
// fma(-q, m, x) is exact.
__device__ __forceinline__ float bal_mod(float x, int l) {
  const float m = (float)kMod[l];
  const float q = rintf(x * (1.0f / m));
  return fmaf(-q, m, x);
}

// ------------------------------------------------------------ 1. max |x| per row
// X(r, k) = X[r * sr + k * sk]; rmax[r] = bits of max_k |X(r, k)| (atomic max
// on the bit pattern of a non-negative double orders like the value, so the
// result does not depend on the order of the workgroups).
__global__ __launch_bounds__(256) void k_crt_rowmax(const double* __restrict__ X, int64_t sr, int64_t sk, int R,
                                                    int K, unsigned long long* __restrict__ rmax) {
  const int t = threadIdx.x;
  const int k0 = blockIdx.y * 256;
  double mx = 0.0;
  int r;
  if (sr == 1) {  // rows contiguous: thread = row, loop over k
    r = blockIdx.x * 256 + t;
    if (r < R)
      for (int k = k0; k < min(K, k0 + 256); ++k) mx = fmax(mx, fabs(X[r + (int64_t)k * sk]));
    if (r < R && mx > 0.0) atomicMax(&rmax[r], (unsigned long long)__double_as_longlong(mx));
  } else {  // k contiguous: a wavefront per row
    const int w = t >> 6, l = t & 63;
    for (int q = 0; q < 64; ++q) {
      r = blockIdx.x * 256 + w * 64 + q;
      if (r >= R) break;
      mx = 0.0;
      for (int k = k0 + l; k < min(K, k0 + 256); k += 64) mx = fmax(mx, fabs(X[(int64_t)r * sr + k]));
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
      if (l == 0 && mx > 0.0) atomicMax(&rmax[r], (unsigned long long)__double_as_longlong(mx));
    }
  }
}

// scale exponent of a row: max * 2^E < 2^beta (0 for an all-zero row)
__device__ __forceinline__ int row_exp(unsigned long long bits, int beta) {
  if (bits == 0ull) return 0;
  return beta - 1 - ilogb(__longlong_as_double((long long)bits));
}

// ------------------------------------------------------------ 2. residues
// Residues of a block of 64 rows x 64 k from (r0, k0): the scaled entries are
// rounded to integers and, for every modulus, a thread writes the 16 balanced
// residues of a quarter row as one 16-byte store (a row's four 64 bytes) at
// out + r * P + l * plane.  |A'| mod m is the sum of its seven bytes times
// 2^(8 b) mod m, two byte dot products (below 2^19, so exact in FP32), then
// bal_mod.  Entries outside (r < R, k < K) are zeros; rows up to Rout are
// written.  The block passes through LDS so that its reads run along whichever
// index is contiguous (RIGHT: k, column stride ld; else the rows) while its
// writes run along k: n = 6000 with nothing deflated, 16 moduli, 1.60 -> 1.09 ms
// for both operands (with each thread reading its own 16 k of a column, 1.9).
constexpr int kSplitLd = 66;  // doubles per row: 16-byte aligned

template <int L, int RIGHT>
__device__ __forceinline__ void split_block(double* __restrict__ tile, const double* __restrict__ X, int64_t ld, int R,
                                            int K, int r0, int k0, int Rout, int beta,
                                            const unsigned long long* __restrict__ rmax, int* __restrict__ rexp,
                                            int8_t* __restrict__ out, int64_t P, int64_t plane) {
  constexpr float kByte = 12582912.0f;  // 3 2^22: the low byte of r + kByte is r's, |r| < 128
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  double x[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const int r = RIGHT ? r0 + 16 * wv + q : r0 + lane, k = RIGHT ? k0 + lane : k0 + 16 * wv + q;
    x[q] = (r < R && k < K) ? (RIGHT ? X[(int64_t)r * ld + k] : X[r + (int64_t)k * ld]) : 0.0;
  }
#pragma unroll
  for (int q = 0; q < 16; ++q) tile[RIGHT ? (16 * wv + q) * kSplitLd + lane : lane * kSplitLd + 16 * wv + q] = x[q];
  __syncthreads();
  const int r = r0 + (t >> 2), kq = 16 * (t & 3);
  if (r >= Rout) return;
  const int E = r < R ? row_exp(rmax[r], beta) : 0;
  if (k0 == 0 && kq == 0 && r < R) rexp[r] = E;
  unsigned int lo[16], hi[16];
  float sg[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const double a = rint(ldexp(tile[(t >> 2) * kSplitLd + kq + e], E));
    sg[e] = a < 0.0 ? -1.0f : 1.0f;
    const unsigned long long u = (unsigned long long)fabs(a);
    lo[e] = (unsigned int)u;
    hi[e] = (unsigned int)(u >> 32);
  }
  out += (int64_t)r * P + k0 + kq;
#pragma unroll
  for (int l = 0; l < L; ++l) {
    unsigned int wd[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      unsigned int v[4];
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const int e = 4 * q + b;
        const unsigned int s = __builtin_amdgcn_udot4(
            lo[e], kTab<L>.pw[RIGHT][l][0], __builtin_amdgcn_udot4(hi[e], kTab<L>.pw[RIGHT][l][1], 0u, false), false);
        v[b] = __float_as_uint(fmaf(bal_mod((float)s, l), sg[e], kByte));
      }
      wd[q] = __builtin_amdgcn_perm(__builtin_amdgcn_perm(v[3], v[2], 0x0c0c0400u),
                                    __builtin_amdgcn_perm(v[1], v[0], 0x0c0c0400u), 0x05040100u);
    }
    *reinterpret_cast<uint4*>(out + l * plane) = make_uint4(wd[0], wd[1], wd[2], wd[3]);
  }
}

// Grid (row block of 64, k block of 64).
template <int L, int RIGHT>
__global__ __launch_bounds__(256) void k_crt_split(const double* __restrict__ X, int64_t ld, int R, int K,
                                                   const unsigned long long* __restrict__ rmax, int beta,
                                                   int8_t* __restrict__ out, int64_t plane, int P, int Rpad,
                                                   int* __restrict__ rexp) {
  __shared__ __attribute__((aligned(16))) double tile[64 * kSplitLd];
  split_block<L, RIGHT>(tile, X, ld, R, K, blockIdx.x * 64, blockIdx.y * 64, Rpad, beta, rmax, rexp, out, P, plane);
}

// ------------------------------------------------------------ 3. residue products
// 256 x 128 output tile per 256-thread workgroup: four wavefronts in 2 x 2,
// each 128 x 64 as 4 x 2 blocks of v_mfma_i32_32x32x32_i8 (the int32 sums of a
// block stay in 16 accumulation registers per lane).  k advances in 64-byte
// stages: the residue tiles of a stage (256 and 128 rows of 64 bytes) are copied from global memory straight
// into LDS by the memory unit (global_load_lds_dwordx4: lane i of an
// instruction lands at the instruction's LDS base + 16 i), into a ring of three
// stage buffers.  A stage has two steps of 32 k; a step's operands are read
// from LDS while the step before is multiplied, and the one barrier of a stage
// lies between its steps, where the next stage must have landed and the
// stage's own buffer is read out: the copies of the stage three ahead go there.
// In LDS the four 16-byte chunks of row r are stored in the order c ^ f(r),
// f(r) = ((r >> 1) ^ (r >> 3)) & 3 (each lane loads the chunk that belongs at
// its slot), so the operand reads of 8 or 16 consecutive lanes, which read the
// same chunk of consecutive rows, fall on distinct banks.  Each lane feeds the
// matrix cores the 16 bytes of chunk 2 kk + (lane >> 5) of row (lane & 31) of
// its A and B blocks: the products sum over all 32 k of a step whichever lanes
// hold which k, as long as A and B agree.  The int32 sums are reduced mod m_l,
// turned around in LDS (a lane holds four rows of a column: stored from there,
// 32 columns an instruction, the stores took as long as 3000 k) and stored as
// balanced int8, column-major (ldr rows).
// Two workgroups share a CU (72 KB of LDS, 184 registers a lane): one's first
// copies, reductions and stores pass while the other multiplies.  n = 6000 with
// nothing deflated (16 moduli): the products of all levels 6.5 -> 3.6 ms, of the
// last one 3.3 -> 2.2 (1.8 POP/s).  256 x 256 tiles, which fill a CU alone:
// 4.3 and 2.5; the stores straight from the accumulators, 32 columns an
// instruction: 6.5 and 2.8.
constexpr int kTile = 256, kTileN = 128, kKs = 64, kRing = 3;
// column stride of a finished tile in LDS: 16-byte reads, and the writes of 16
// consecutive columns fall on distinct banks
constexpr int kOutLd = kTile + 16;

struct CrtSmem {
  union {
    struct {
      int8_t A[kRing][kTile * kKs];
      int8_t B[kRing][kTileN * kKs];
    };
    int8_t out[kTileN * kOutLd];
  };
};

__device__ __forceinline__ int crt_swz(int r) { return ((r >> 1) ^ (r >> 3)) & 3; }

// s_waitcnt for at most N vector-memory operations in flight and no LDS ones
// (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4 at its maximum,
// lgkmcnt 11:8)
template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

__device__ __forceinline__ void copy_to_lds(const int8_t* from, int8_t* to) {
  __builtin_amdgcn_global_load_lds(from, to, 16, 0, 0);
}

// a lane's value that the compiler cannot trace back: it would otherwise keep
// every lane's addresses of all copies, reads and stores across the k loop
__device__ __forceinline__ int hidden(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// One 256 x 128 tile: A rows row0.., B^T rows col0.. (both k contiguous,
// stride P, nk stages; the rows up to 255 (A) and 127 (B) past the tile's
// first ones must be readable), output (i, j) mod m_l at C[j ldr + i] for
// i < M, j < N (tile-relative bounds; C and ldr multiples of 4, and the bytes
// after row M - 1 up to a multiple of 4 are written too).
__device__ __forceinline__ void crt_tile(CrtSmem& sm, const int8_t* __restrict__ A, const int8_t* __restrict__ B,
                                         int P, int nk, int M, int N, int l, int8_t* __restrict__ C, int64_t ldr) {
  constexpr int BB = kTileN / 64;  // 32 x 32 blocks along a wavefront's columns
  constexpr int kCopies = 4 + BB;  // per thread and stage
  const int t = hidden(threadIdx.x);
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6), ln = t & 63;
  const int wm = wv & 1, wn = wv >> 1;
  // slot q * 256 + t of a stage: row 64 q + t / 4, position t % 4, holding
  // chunk position ^ f(row) of that row (f is the same for all q)
  const int64_t from = (int64_t)(t >> 2) * P + 16 * ((t & 3) ^ crt_swz(t >> 2));
  const int8_t* ga = A + from;
  const int8_t* gb = B + from;
  // the copies of stage s into ring buffer s % kRing; the LDS base of an
  // instruction is uniform over the wavefront
  auto issue = [&](int s, int buf) {
    const int k0 = s * kKs;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      copy_to_lds(ga + ((int64_t)(64 * q) * P + k0), &sm.A[buf][16 * (q * 256 + wv * 64)]);
#pragma unroll
    for (int q = 0; q < BB; ++q)
      copy_to_lds(gb + ((int64_t)(64 * q) * P + k0), &sm.B[buf][16 * (q * 256 + wv * 64)]);
  };
  v16i acc[4][BB];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < BB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0;
  const int lr = ln & 31, lh = ln >> 5;
  // f(32 a + lr) = f(lr): a lane's reads of a step are 2 KB apart
  const int chunk[2] = {lr * kKs + 16 * (lh ^ crt_swz(lr)), lr * kKs + 16 * ((2 + lh) ^ crt_swz(lr))};
  struct Step {
    v4i a[4], b[BB];
  };
  auto read = [&](Step& f, int buf, int kk) {
    const int8_t* pa = &sm.A[buf][wm * 128 * kKs + chunk[kk]];
    const int8_t* pb = &sm.B[buf][wn * (kTileN / 2) * kKs + chunk[kk]];
#pragma unroll
    for (int a = 0; a < 4; ++a) f.a[a] = *reinterpret_cast<const v4i*>(pa + a * 32 * kKs);
#pragma unroll
    for (int b = 0; b < BB; ++b) f.b[b] = *reinterpret_cast<const v4i*>(pb + b * 32 * kKs);
  };
  auto multiply = [&](const Step& f) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < BB; ++b)
        acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(f.a[a], f.b[b], acc[a][b], 0, 0, 0);
  };
  // the previous tile's readers are done with every ring buffer
  __syncthreads();
#pragma unroll
  for (int s = 0; s < kRing; ++s)
    if (s < nk) issue(s, s);
  if (nk >= kRing) wait_vm<(kRing - 1) * kCopies>();
  else wait_vm<0>();
  __builtin_amdgcn_s_barrier();
  Step f0, f1;
  read(f0, 0, 0);
  int buf = 0;
  for (int s = 0; s < nk - 1; ++s) {
    read(f1, buf, 1);
    multiply(f0);
    // stage s + 1 has landed (those after it may still fly); this wavefront
    // has read stage s out.  After the barrier that holds for all of them.
    if (s + kRing - 1 < nk) wait_vm<(kRing - 2) * kCopies>();
    else wait_vm<0>();
    __builtin_amdgcn_s_barrier();
    if (s + kRing < nk) issue(s + kRing, buf);
    buf = buf == kRing - 1 ? 0 : buf + 1;
    read(f0, buf, 0);
    multiply(f1);
  }
  read(f1, buf, 1);
  multiply(f0);
  multiply(f1);
  // D[i][j] of a 32 x 32 block: lane j + 32 h, register r holds row
  // 8 (r / 4) + 4 h + r % 4: four consecutive rows per register quad.  The sum
  // x mod m: 2^52 + 2^31 + x is put together from its bits, the quotient is
  // rounded by adding 3 2^51, and the fused remainder leaves 2^52 + 2^31 + r,
  // whose low byte is r's (x/m is never within 1/(2m) of a half-integer).
  constexpr double kBias = 0x1p52 + 0x1p31, kRound = 0x1.8p52;
  const int te = hidden(t), er = te & 31, eh = (te >> 5) & 1;
  const double m = (double)kMod[l], im = 1.0 / m;
  __syncthreads();  // every wavefront has read the last stage out
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < BB; ++b)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        unsigned int v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double x = __hiloint2double(0x43300000, acc[a][b][4 * g + q] ^ (int)0x80000000u);
          const double quo = fma(x - kBias, im, kRound) - kRound;
          v[q] = (unsigned int)__double2loint(fma(-quo, m, x));
        }
        *reinterpret_cast<unsigned int*>(
            &sm.out[(wn * (kTileN / 2) + b * 32 + er) * kOutLd + wm * 128 + a * 32 + 8 * g + 4 * eh]) =
            __builtin_amdgcn_perm(__builtin_amdgcn_perm(v[3], v[2], 0x0c0c0400u),
                                  __builtin_amdgcn_perm(v[1], v[0], 0x0c0c0400u), 0x05040100u);
      }
  __syncthreads();
  // a column's rows leave as one run, 16 bytes per lane, to the word that
  // holds row M - 1
  const int orow = 16 * (te & 15);
  if (orow >= M) return;
#pragma unroll 4
  for (int c = te >> 4; c < kTileN; c += 16) {
    if (c >= N) break;
    const uint4 x = *reinterpret_cast<const uint4*>(&sm.out[c * kOutLd + orow]);
    unsigned int* dst = reinterpret_cast<unsigned int*>(C + (int64_t)c * ldr + orow);
    if (orow + 12 < M) {
      *reinterpret_cast<CrtWords*>(dst) = CrtWords{x.x, x.y, x.z, x.w};
    } else {
      dst[0] = x.x;
      if (orow + 4 < M) dst[1] = x.y;
      if (orow + 8 < M) dst[2] = x.z;
    }
  }
}

// Grid: x = output tiles, z = modulus.  Residues of the products,
// column-major (ldr rows).
__global__ __launch_bounds__(256, 2) void k_crt_gemm(const int8_t* __restrict__ RA, const int8_t* __restrict__ RB,
                                                     int64_t planeA, int64_t planeB, int P, int M, int N,
                                                     int8_t* __restrict__ RC, int64_t planeC, int ldr) {
  __shared__ __attribute__((aligned(16))) CrtSmem sm;
  const int l = blockIdx.z;
  int tm, tn;
  // consecutive workgroups go to the 8 XCDs in turn: those of one share panels
  gemm128_place(blockIdx.x, 8, (M + kTile - 1) / kTile, (N + kTileN - 1) / kTileN, tm, tn);
  const int row0 = tm * kTile, col0 = tn * kTileN;
  crt_tile(sm, RA + l * planeA + (int64_t)row0 * P, RB + l * planeB + (int64_t)col0 * P, P, P / kKs, M - row0,
               N - col0, l, RC + l * planeC + (int64_t)col0 * ldr + row0, ldr);
}

// ------------------------------------------------------------ 4. rebuild
// x 2^e (x in 128-bit two's complement, |x| < 2^126) rounded once to FP64 (to
// nearest, ties to even): an exact product of integers comes out bit for bit.
__device__ __forceinline__ double round_i128(long long hi, unsigned long long lo, int e) {
  const bool neg = hi < 0;
  unsigned long long uh = (unsigned long long)hi, ul = lo;
  if (neg) {  // magnitude
    ul = ~ul + 1ull;
    uh = ~uh + (ul == 0ull ? 1ull : 0ull);
  }
  if (uh == 0ull && ul == 0ull) return 0.0;
  unsigned long long t;
  bool sticky;
  if (uh != 0ull) {
    const int lz = __clzll((long long)uh);
    t = lz ? (uh << lz) | (ul >> (64 - lz)) : uh;
    sticky = lz ? (ul << lz) != 0ull : ul != 0ull;
    e += 64 - lz;
  } else {
    const int lz = __clzll((long long)ul);
    t = ul << lz;
    sticky = false;
    e -= lz;
  }
  // |x| 2^e = (t + a fraction below its last bit) 2^e; keep the top 53 bits of t
  unsigned long long mant = t >> 11;
  const unsigned int rem = (unsigned int)(t & 0x7FFull);
  if (rem > 0x400u || (rem == 0x400u && (sticky || (mant & 1ull)))) ++mant;
  const double v = ldexp((double)mant, e + 11);
  return neg ? -v : v;
}

// The integer x, |x| <= (M - 1)/2, with x = sum_l v_l (M/m_l) mod M, times 2^e;
// byte l of v holds v_l (zero past L).  Each base-256 digit of the sum is a dot
// product of 16 bytes with the constants' digits, below 2^18 in magnitude; the
// digits are put together in 64-bit words of weight 2^(32 j), the multiple of
// M is taken off and the carries are passed on.  That multiple is the rounded
// quotient in FP32, exact but where x/M is within 2^-18 of a half, which the
// comparison with (M - 1)/2 sets right.  About 190 operations an element where
// Garner's mixed radix takes 120 dependent modular steps (about 850): the
// rebuild of n = 6000 with nothing deflated 2.55 -> 0.77 ms.
template <int L>
__device__ __forceinline__ double rebuild(const unsigned int (&v)[4], int e) {
  constexpr CrtTables<L> T = kTab<L>;
  int t[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    int d[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int b = 2 * k + h;
      d[h] = 0;
      if (b < kDigits) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (T.dig[b][q]) d[h] = __builtin_amdgcn_sdot4((int)v[q], (int)T.dig[b][q], d[h], false);
      }
    }
    t[k] = d[0] + 256 * d[1];
  }
  float qf = 0.0f;
#pragma unroll
  for (int k = 3; k < 8; ++k) qf = fmaf((float)t[k], T.part[k], qf);
  const int q = -(int)rintf(qf);
  long long u[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    u[j] = (long long)q * T.mlimb[j] + ((long long)t[2 * j + 1] * 65536 + t[2 * j]);
#pragma unroll
  for (int j = 0; j < 3; ++j) u[j + 1] += u[j] >> 32;
  unsigned long long lo = (unsigned long long)(unsigned int)u[0] | ((unsigned long long)(unsigned int)u[1] << 32);
  long long hi = (long long)((unsigned long long)(unsigned int)u[2] | ((unsigned long long)(unsigned int)u[3] << 32));
  if (hi >= T.hhi || hi <= -T.hhi - 1) {
    const __int128 x = ((__int128)hi << 64) | lo, half = ((__int128)T.hhi << 64) | T.hlo,
                   M = ((__int128)T.mhi << 64) | T.mlo;
    const __int128 z = x > half ? x - M : (x < -half ? x + M : x);
    hi = (long long)(z >> 64);
    lo = (unsigned long long)z;
  }
  return round_i128(hi, lo, e);
}

// Rows row0 .. row0 + 255 of one output column, a wavefront: lane t rebuilds
// rows row0 + 4 t + 0..3, whose residues are one word per plane (col and planeC
// multiples of 4), and the values are turned around in LDS (tile, the
// wavefront's own) so that each store covers 512 contiguous bytes.  rows: the
// column's end.
template <int L>
__device__ __forceinline__ void rebuild_rows(const int8_t* __restrict__ col, int64_t planeC, int row0, int rows,
                                             const int* __restrict__ ea, int eb, double* __restrict__ dst,
                                             double* tile) {
  const int lane = threadIdx.x & 63;
  const int i0 = row0 + 4 * lane;
  unsigned int r[16];
#pragma unroll
  for (int l = 0; l < 16; ++l) r[l] = 0u;
  int ee[4];
  if (i0 < rows) {
#pragma unroll
    for (int l = 0; l < L; ++l) r[l] = *reinterpret_cast<const unsigned int*>(col + l * planeC + i0);
  }
#pragma unroll
  for (int x = 0; x < 4; ++x) ee[x] = ea[min(i0 + x, rows - 1)];
  unsigned int v[4][4];  // [row][planes 4 g .. 4 g + 3]
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const unsigned int a = __builtin_amdgcn_perm(r[4 * g + 1], r[4 * g], 0x05010400u),
                       b = __builtin_amdgcn_perm(r[4 * g + 3], r[4 * g + 2], 0x05010400u),
                       c = __builtin_amdgcn_perm(r[4 * g + 1], r[4 * g], 0x07030602u),
                       d = __builtin_amdgcn_perm(r[4 * g + 3], r[4 * g + 2], 0x07030602u);
    v[0][g] = __builtin_amdgcn_perm(b, a, 0x05040100u);
    v[1][g] = __builtin_amdgcn_perm(b, a, 0x07060302u);
    v[2][g] = __builtin_amdgcn_perm(d, c, 0x05040100u);
    v[3][g] = __builtin_amdgcn_perm(d, c, 0x07060302u);
  }
  double out[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) out[x] = rebuild<L>(v[x], -(ee[x] + eb));
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int x = 0; x < 4; x += 2)
    *reinterpret_cast<double2*>(&tile[4 * lane + x]) = make_double2(out[x], out[x + 1]);
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const int i = row0 + 64 * x + lane;
    if (i < rows) dst[i] = tile[64 * x + lane];
  }
  __builtin_amdgcn_wave_barrier();
}

// A wavefront per 256 rows of a column, scaled by 2^-(E_r + E_c).
template <int L>
__global__ __launch_bounds__(256) void k_crt_combine(const int8_t* __restrict__ RC, int64_t planeC, int ldr, int M,
                                                     int N, const int* __restrict__ ea, const int* __restrict__ eb,
                                                     double* __restrict__ C, int64_t ldc) {
  __shared__ __attribute__((aligned(16))) double tile[4][256];
  const int wv = threadIdx.x >> 6;
  const int chunks = (M + 255) / 256;
  const int64_t u = (int64_t)blockIdx.x * 4 + wv;
  if (u >= (int64_t)chunks * N) return;
  const int col = (int)(u / chunks), row0 = (int)(u % chunks) * 256;
  rebuild_rows<L>(RC + (int64_t)col * ldr, planeC, row0, M, ea, eb[col], C + (int64_t)col * ldc, tile[wv]);
}

// ------------------------------------------------------------ vector update of a merge level
// Geometry of one half-side of a merge's update (sub: 0 U rows [0,k), 1 U
// rows [k,m), 2 V rows [0,k), 3 V rows [k,m+s)): left operand = gathered
// kept columns [kb, kb+K) of those rows, right operand = rows [kb, kb+K) of
// the N x N vectors of M.
struct CrtHalf {
  int rows, kb, K, rowoff, isV, bottom;
  int crow;  // first row in the planes of the products
};
// In those planes a merge has its columns to itself, so its top half starts
// at row 0 and its bottom half at the next multiple of 4 (whole words).  The
// rows fit the stride, n + 1 rounded up to 16: k is half of m, so the widest
// merge, m = n and s = 0, ends by row n + 3, and by n + 1 if n mod 16 is 14 or 15.
__device__ inline CrtHalf crt_half(const NodeDesc& nd, const NodeState& st, int sub) {
  CrtHalf h;
  h.isV = sub >= 2;
  h.bottom = sub & 1;
  h.rows = h.bottom ? (h.isV ? nd.m + nd.s - nd.k : nd.m - nd.k) : nd.k;
  h.kb = h.bottom ? st.n1 : 0;
  const int ke = h.bottom ? st.N : st.n1 + 1 + st.n2;
  h.K = ke - h.kb;
  h.rowoff = h.bottom ? nd.k : 0;
  h.crow = h.bottom ? (nd.k + 3) & ~3 : 0;
  return h;
}

// Zero the maxima of the merges that take the split products.  Grid (node, 1, sub).
__global__ __launch_bounds__(256) void k_crt_lvl_clear(const NodeDesc* __restrict__ nodes, Work w) {
  const NodeDesc nd = nodes[blockIdx.x];
  const NodeState st = w.st[nd.id];
  if (st.N < w.oz.min_n) return;
  const CrtHalf h = crt_half(nd, st, blockIdx.z);
  unsigned long long* am = w.crt.amax[h.isV] + nd.r0 + h.rowoff;
  for (int i = threadIdx.x; i < h.rows; i += 256) am[i] = 0ull;
  unsigned long long* bm = (h.bottom ? w.crt.bbmax[h.isV] : w.crt.btmax[h.isV]) + nd.r0;
  for (int c = threadIdx.x; c < st.N; c += 256) bm[c] = 0ull;
}

// Largest |entry| per row of the left operands: grid (node, row block of 256
// x k chunk of 256, sub), a thread per row.
__global__ __launch_bounds__(256) void k_crt_lvl_amax(const NodeDesc* __restrict__ nodes, int kchunks, Work w) {
  const NodeDesc nd = nodes[blockIdx.x];
  const NodeState st = w.st[nd.id];
  if (st.N < w.oz.min_n) return;
  const CrtHalf h = crt_half(nd, st, blockIdx.z);
  const int rb = blockIdx.y / kchunks, kc = blockIdx.y % kchunks;
  const int row = rb * 256 + threadIdx.x, k0 = kc * 256;
  if (row >= h.rows || k0 >= h.K) return;
  const int64_t ld = nd.ld;
  const double* G = (h.isV ? w.ctl->io.VT : w.ctl->io.U) + nd.mat_off + (nd.r0 + h.rowoff + row) + (int64_t)(nd.r0 + h.kb) * ld;
  double mx = 0.0;
  const int ke = min(h.K, k0 + 256);
#pragma unroll 16
  for (int k = k0; k < ke; ++k) mx = fmax(mx, fabs(G[(int64_t)k * ld]));
  if (mx > 0.0) atomicMax(&w.crt.amax[h.isV][nd.r0 + h.rowoff + row], (unsigned long long)__double_as_longlong(mx));
}

// Largest |entry| per column of the right operands: grid (node, column block
// of 64 x k chunk of 256, sub); a wavefront per column.
__global__ __launch_bounds__(256) void k_crt_lvl_bmax(const NodeDesc* __restrict__ nodes, int kchunks, Work w) {
  const NodeDesc nd = nodes[blockIdx.x];
  const NodeState st = w.st[nd.id];
  if (st.N < w.oz.min_n) return;
  const CrtHalf h = crt_half(nd, st, blockIdx.z);
  const int cb = blockIdx.y / kchunks, kc = blockIdx.y % kchunks;
  const int k0 = kc * 256;
  if (k0 >= h.K) return;
  const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
  const int64_t ld = nd.ld;
  const double* Mv = (h.isV ? w.VM : w.UM) + nd.mat_off + (nd.r0 + h.kb);
  unsigned long long* bm = (h.bottom ? w.crt.bbmax[h.isV] : w.crt.btmax[h.isV]) + nd.r0;
  const int ke = min(h.K, k0 + 256);
  // four columns at a time: 16 loads in flight
  for (int q = 0; q < 16; q += 4) {
    const int c0 = cb * 64 + wv * 16 + q;
    if (c0 >= st.N) break;
    double mx[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      mx[x] = 0.0;
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        const int k = k0 + ln + 64 * y;
        if (c0 + x < st.N && k < ke) mx[x] = fmax(mx[x], fabs(Mv[k + (int64_t)(nd.r0 + c0 + x) * ld]));
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int x = 0; x < 4; ++x) mx[x] = fmax(mx[x], __shfl_xor(mx[x], o, 64));
#pragma unroll
    for (int x = 0; x < 4; ++x)
      if (ln == 0 && mx[x] > 0.0) atomicMax(&bm[c0 + x], (unsigned long long)__double_as_longlong(mx[x]));
  }
}

// Residues of the left operands (RIGHT 0: rows contiguous) and of the right
// ones (1: columns of the vectors of M, k contiguous): grid (node, row block of
// 64 x k block of 64, sub).
template <int L, int RIGHT>
__global__ __launch_bounds__(256) void k_crt_lvl_split(const NodeDesc* __restrict__ nodes, int kblocks, int beta,
                                                       Work w) {
  __shared__ __attribute__((aligned(16))) double tile[64 * kSplitLd];
  const NodeDesc nd = nodes[blockIdx.x];
  const NodeState st = w.st[nd.id];
  if (st.N < w.oz.min_n) return;
  const CrtHalf h = crt_half(nd, st, blockIdx.z);
  const int r0 = (blockIdx.y / kblocks) * 64, k0 = (blockIdx.y % kblocks) * 64;
  const int R = RIGHT ? st.N : h.rows;
  if (r0 >= R || k0 >= crt_kpad(h.K)) return;
  const int64_t ld = nd.ld;
  if constexpr (RIGHT) {
    const double* Mv = (h.isV ? w.VM : w.UM) + nd.mat_off + (nd.r0 + h.kb) + (int64_t)nd.r0 * ld;
    const unsigned long long* bm = h.bottom ? w.crt.bbmax[h.isV] : w.crt.btmax[h.isV];
    int* Eb = h.bottom ? w.crt.Ebb[h.isV] : w.crt.Ebt[h.isV];
    int8_t* out = (h.bottom ? w.crt.Bb[h.isV] : w.crt.Bt[h.isV]) + (int64_t)nd.r0 * w.crt.P;
    split_block<L, 1>(tile, Mv, ld, R, h.K, r0, k0, R, beta, bm + nd.r0, Eb + nd.r0, out, w.crt.P, w.crt.planeB);
  } else {
    const int prow = nd.r0 + h.rowoff;
    const double* G = (h.isV ? w.ctl->io.VT : w.ctl->io.U) + nd.mat_off + prow + (int64_t)(nd.r0 + h.kb) * ld;
    split_block<L, 0>(tile, G, ld, R, h.K, r0, k0, R, beta, w.crt.amax[h.isV] + prow, w.crt.Ea[h.isV] + prow,
                      w.crt.A[h.isV] + (int64_t)prow * w.crt.P, w.crt.P, w.crt.planeA);
  }
}

// Residue products: grid (node + nnodes * tile, 1, sub * L + modulus), a tile
// each.
template <int L>
__global__ __launch_bounds__(256, 2) void k_crt_lvl_gemm(const NodeDesc* __restrict__ nodes, int nnodes, Work w) {
  __shared__ __attribute__((aligned(16))) CrtSmem sm;
  const NodeDesc nd = nodes[blockIdx.x % nnodes];
  const NodeState st = w.st[nd.id];
  if (st.N < w.oz.min_n) return;
  const int sub = blockIdx.z / L, l = blockIdx.z % L;
  const CrtHalf h = crt_half(nd, st, sub);
  // in scalar registers: the loop has none of the others to spare
  auto scalar = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  const int P = w.crt.P, rows = scalar(h.rows), N = scalar(st.N), nk = scalar(crt_kpad(h.K) / kKs), r0 = scalar(nd.r0),
            rowoff = scalar(h.rowoff);
  const int tiles_m = (rows + kTile - 1) / kTile, tiles_n = (N + kTileN - 1) / kTileN;
  const int tile = blockIdx.x / nnodes;
  if (tile >= tiles_m * tiles_n) return;
  // workgroups of a node Q tiles apart share an XCD (the grid is a multiple of 8 wide)
  int tm, tn;
  gemm128_place(tile, 8 / min(8, nnodes & -nnodes), tiles_m, tiles_n, tm, tn);
  const int row0 = tm * kTile, col0 = tn * kTileN;
  const int side = sub >= 2;
  const int8_t* A = w.crt.A[side] + l * w.crt.planeA + (int64_t)(r0 + rowoff + row0) * P;
  const int8_t* B = ((sub & 1) ? w.crt.Bb[side] : w.crt.Bt[side]) + l * w.crt.planeB + (int64_t)(r0 + col0) * P;
  int8_t* C = w.crt.C[side] + l * w.crt.planeC + (int64_t)(r0 + col0) * w.crt.ldr + scalar(h.crow) + row0;
  crt_tile(sm, A, B, P, nk, rows - row0, N - col0, l, C, w.crt.ldr);
}

// Rebuild into the kept values' physical columns: grid (node, y, sub), a
// wavefront per 256 rows of a column.
template <int L>
__global__ __launch_bounds__(256) void k_crt_lvl_combine(const NodeDesc* __restrict__ nodes, Work w) {
  __shared__ __attribute__((aligned(16))) double tile[4][256];
  const NodeDesc nd = nodes[blockIdx.x];
  const NodeState st = w.st[nd.id];
  if (st.N < w.oz.min_n) return;
  const CrtHalf h = crt_half(nd, st, blockIdx.z);
  const int64_t vo = nd.vec_off + nd.r0;
  double* dst = (h.isV ? w.Vw : w.Uw) + nd.mat_off + nd.r0 + h.rowoff;
  const int* Ea = w.crt.Ea[h.isV] + nd.r0 + h.rowoff;
  const int* Eb = (h.bottom ? w.crt.Ebb[h.isV] : w.crt.Ebt[h.isV]) + nd.r0;
  const int8_t* C = w.crt.C[h.isV] + (int64_t)nd.r0 * w.crt.ldr + h.crow;
  const int wv = threadIdx.x >> 6;
  const int chunks = (h.rows + 255) / 256;
  const int units = chunks * st.N;
  for (int u = (int)blockIdx.y * 4 + wv; u < units; u += (int)gridDim.y * 4) {
    const int c = u / chunks, row0 = u % chunks * 256;
    rebuild_rows<L>(C + (int64_t)c * w.crt.ldr, w.crt.planeC, row0, h.rows, Ea, Eb[c],
                    dst + (int64_t)w.scol[vo + c] * nd.ld, tile[wv]);
  }
}

template <int L>
void launch_crt_level(const NodeDesc* nodes, int nnodes, int max_m, const Work& w, hipStream_t st) {
  const int rmax = max_m + 1;                  // rows of the largest half-side, bounded
  const int kmax = max_m;                      // kept values bound the product depth
  const int beta = crt_beta(L, crt_kpad(kmax));
  const int kc256 = (kmax + 255) / 256, kb64 = crt_kpad(kmax) / 64;
  hipLaunchKernelGGL(k_crt_lvl_clear, dim3(nnodes, 1, 4), dim3(256), 0, st, nodes, w);
  hipLaunchKernelGGL(k_crt_lvl_amax, dim3(nnodes, ((rmax + 255) / 256) * kc256, 4), dim3(256), 0, st, nodes, kc256,
                     w);
  hipLaunchKernelGGL(k_crt_lvl_bmax, dim3(nnodes, ((kmax + 63) / 64) * kc256, 4), dim3(256), 0, st, nodes, kc256, w);
  hipLaunchKernelGGL((k_crt_lvl_split<L, 0>), dim3(nnodes, ((rmax + 63) / 64) * kb64, 4), dim3(256), 0, st, nodes, kb64,
                     beta, w);
  hipLaunchKernelGGL((k_crt_lvl_split<L, 1>), dim3(nnodes, ((kmax + 63) / 64) * kb64, 4), dim3(256), 0, st, nodes, kb64,
                     beta, w);
  const unsigned slots = (((rmax + kTile - 1) / kTile) * ((kmax + kTileN - 1) / kTileN) + 7) & ~7;  // of any half-side
  hipLaunchKernelGGL(k_crt_lvl_gemm<L>, dim3(nnodes * slots, 1, 4 * L), dim3(256), 0, st, nodes, nnodes, w);
  const int64_t runs = (int64_t)((rmax + 255) / 256) * kmax;
  const int ey = (int)std::min<int64_t>((runs + 3) / 4, std::max(1, 8192 / std::max(1, nnodes)));
  hipLaunchKernelGGL(k_crt_lvl_combine<L>, dim3(nnodes, ey, 4), dim3(256), 0, st, nodes, w);
}

template <int L>
void gemm_crt_plain_L(int M, int N, int K, const double* A, int lda, const double* B, int ldb, double* C, int ldc,
                      const CrtBuffers& b, hipStream_t st) {
  const int P = crt_kpad(K);
  const int Mp = crt_rowpad(M), Np = crt_rowpad(N);
  const int beta = crt_beta(L, P);
  (void)hipMemsetAsync(b.amax, 0, sizeof(unsigned long long) * M, st);
  (void)hipMemsetAsync(b.bmax, 0, sizeof(unsigned long long) * N, st);
  // A: rows contiguous (column-major); B^T rows = columns of B, k contiguous
  k_crt_rowmax<<<dim3((M + 255) / 256, (K + 255) / 256), 256, 0, st>>>(A, 1, lda, M, K, b.amax);
  k_crt_rowmax<<<dim3((N + 255) / 256, (K + 255) / 256), 256, 0, st>>>(B, ldb, 1, N, K, b.bmax);
  const int64_t planeA = (int64_t)Mp * P, planeB = (int64_t)Np * P;
  k_crt_split<L, 0><<<dim3(Mp / 64, P / 64), 256, 0, st>>>(A, lda, M, K, b.amax, beta, b.ra, planeA, P, Mp, b.ea);
  k_crt_split<L, 1><<<dim3(Np / 64, P / 64), 256, 0, st>>>(B, ldb, N, K, b.bmax, beta, b.rb, planeB, P, Np, b.eb);
  const int ldr = Mp;
  const int64_t planeC = (int64_t)Mp * N;
  const int tiles = (Mp / kTile) * ((N + kTileN - 1) / kTileN);
  k_crt_gemm<<<dim3(tiles, 1, L), 256, 0, st>>>(b.ra, b.rb, planeA, planeB, P, M, N, b.rc, planeC, ldr);
  const int64_t runs = (int64_t)((M + 255) / 256) * N;
  k_crt_combine<L><<<dim3((unsigned)((runs + 3) / 4)), 256, 0, st>>>(b.rc, planeC, ldr, M, N, b.ea, b.eb, C,
                                                                          ldc);
}

}  // namespace

int crt_beta(int L, int P) {
  double lg = 0.0;
  for (int l = 0; l < L; ++l) lg += std::log2((double)kMod[l]);
  int lk = 0;
  while ((1 << lk) < P) ++lk;
  // K 2^(2 beta) <= (M - 1) / 2 with a little room for the log2 rounding;
  // at most 55, so that |A'| <= 2^55 fits the seven bytes split_block takes
  return std::min(kCrtMaxBeta, (int)std::floor((lg - 1.0 - lk - 1e-9) / 2.0));
}

bool crt_supported(int L) { return L >= kCrtMinMod && L <= kCrtMaxMod; }

size_t crt_plain_bytes(int L, int M, int N, int K, CrtBuffers* b) {
  const int P = crt_kpad(K), Mp = crt_rowpad(M), Np = crt_rowpad(N);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off += (bytes + 255) & ~size_t(255);
    return o;
  };
  const size_t ora = take((size_t)L * Mp * P), orb = take((size_t)L * Np * P), orc = take((size_t)L * Mp * N);
  const size_t oam = take(8 * (size_t)std::max(M, 1)), obm = take(8 * (size_t)std::max(N, 1));
  const size_t oea = take(4 * (size_t)std::max(M, 1)), oeb = take(4 * (size_t)std::max(N, 1));
  if (b) {
    char* base = (char*)b->base;
    b->ra = (int8_t*)(base + ora);
    b->rb = (int8_t*)(base + orb);
    b->rc = (int8_t*)(base + orc);
    b->amax = (unsigned long long*)(base + oam);
    b->bmax = (unsigned long long*)(base + obm);
    b->ea = (int*)(base + oea);
    b->eb = (int*)(base + oeb);
  }
  return off;
}

void launch_update_crt(const NodeDesc* nodes, int nnodes, int max_m, const Work& w, hipStream_t st) {
  if (nnodes <= 0 || max_m < w.oz.min_n) return;
  switch (w.crt.L) {
    case 13: launch_crt_level<13>(nodes, nnodes, max_m, w, st); break;
    case 14: launch_crt_level<14>(nodes, nnodes, max_m, w, st); break;
    case 15: launch_crt_level<15>(nodes, nnodes, max_m, w, st); break;
    case 16: launch_crt_level<16>(nodes, nnodes, max_m, w, st); break;
    default: break;
  }
}

void launch_gemm_crt_plain(int L, int M, int N, int K, const double* A, int lda, const double* B, int ldb, double* C,
                           int ldc, const CrtBuffers& b, hipStream_t st) {
  switch (L) {
    case 13: gemm_crt_plain_L<13>(M, N, K, A, lda, B, ldb, C, ldc, b, st); break;
    case 14: gemm_crt_plain_L<14>(M, N, K, A, lda, B, ldb, C, ldc, b, st); break;
    case 15: gemm_crt_plain_L<15>(M, N, K, A, lda, B, ldb, C, ldc, b, st); break;
    case 16: gemm_crt_plain_L<16>(M, N, K, A, lda, B, ldb, C, ldc, b, st); break;
    default: break;
  }
}

}  // namespace bdc
