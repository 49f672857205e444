// FP64-accurate filter products on the INT8 matrix cores (an integer
// modular emulation of a floating-point matrix product: Ozaki, Uchino and
// Imamura's "Ozaki scheme II").
//
// C = H X with H (n x n) and X (n x k) in FP64.  Each row i of H is scaled by
// 2^sigma_i and each column j of X by 2^tau_j and rounded to integers of at
// most pa and pb bits; the integer product is then exact modulo each of N
// pairwise coprime moduli m_t <= 256, whose residues fit int8: one INT8
// GEMM with exact INT32 accumulation per modulus.  Chinese remaindering
// (Garner's mixed-radix form with balanced digits) recovers the integer
// product, exact because its magnitude stays below M / 2, M = prod m_t;
// scaling back gives C with the rounding error of the integer forms only
// (2^-pa of a row's largest entry, 2^-pb of a column's), which with N = 14
// moduli is about 2^-46: the accuracy class of an FP64 product.
//
// Complex products use Gauss's three real products (Re H + Im H)(Re X +
// Im X), Re H Re X, Im H Im X, combined in residue space, so the real and
// imaginary parts are each reconstructed once.  H is Hermitian: row i of H is
// the conjugate of column i, which makes the conversion of H read contiguous
// memory.  The residue planes of H are built once per solve; those of the
// block at every step.  The N (complex: 3N) INT8 products of a step are one
// launch, whose epilogue reduces each INT32 product modulo its plane's modulus
// to a byte; the reconstruction kernel applies the Chebyshev step of Eq. (3)
// (and the defect-correction term) on the way out.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <utility>

namespace chase {
namespace {

constexpr int TPB = 256;
// pairwise coprime moduli <= 256 (256 = 2^8; 255 = 3 5 17; 253 = 11 23;
// 247 = 13 19; the rest prime), largest first
constexpr int kModuli[kCrtMaxModuli] = {256, 255, 253, 251, 247, 241, 239, 233,
                                        229, 227, 223, 211, 199, 197, 193, 191};

// balanced residue of an integer-valued double |x| < 2^53 modulo m
__device__ __forceinline__ int bres(double x, int m, double minv) {
  const double q = rint(x * minv);
  int r = (int)fma(-q, (double)m, x);  // exact: the result is small
  if (r > (m - 1) / 2) r -= m;
  if (r < -(m / 2)) r += m;
  return r;
}

// x mod m in [0, m) for |x| < 2^31 (int32 GEMM output)
__device__ __forceinline__ int ures32(int x, int m, double minv) {
  const double q = floor((double)x * minv);
  int r = (int)((double)x - q * (double)m);
  if (r < 0) r += m;
  if (r >= m) r -= m;
  return r;
}

// exponent e with |v| < 2^e (frexp), 0 for v == 0
__device__ __forceinline__ int exp2_above(double v) {
  int e = 0;
  if (v > 0.0) (void)frexp(v, &e);
  return e;
}

// Plane layout: rows of H's planes and columns of the block's are contiguous
// along K and padded with zeros to ld(n) = n rounded up to 16 bytes, so that
// every 16-byte piece is aligned and lies within one row.
constexpr int64_t plane_ld(int64_t n) { return (n + 15) / 16 * 16; }

// ------------------------------------------------------------------ INT8 products
// Residues of the P products C_p = A_p B_p: A_p the n x n plane of H (row-major),
// B_p the n x cols plane of the block (column-major); out[p][j ld + i] = C_p(i,
// j) mod m_p in [0, m_p), one byte (a quarter of the INT32 products' bytes, here
// and where the reconstruction reads them).
//
// Eight waves, 4 x 2 of 64 rows x 16 FN columns, share a tile of 256 rows x 32
// FN columns; a wave's part is 4 x FN MFMAs of 16 x 16 x 64.  Both operands go
// global -> LDS by the direct LDS loads (16 bytes a lane, no registers) in K
// chunks of 128 bytes, into GST stages.  A row's eight pieces are XOR-swizzled
// so that the 16 rows a read touches fall into different banks.  Fragment f of
// a wave holds rows 16 (l / 4) + 4 f + l % 4 (l = lane % 16): then the four
// fragments' accumulators of a lane are 16 consecutive rows of one column, and
// their residues go out as one 16-byte store.
//
// Bound by the rate at which a compute unit's tiles arrive (the planes of H
// are beyond the caches), so the largest tile wins: 14 moduli, complex, n=4000
// with 260 columns 274 us (1275 TOP/s; 480 us the library's batched GEMM, which
// also wrote INT32), n=20000 with 1300 23.8 ms (1833 TOP/s).  Slower: half as
// deep chunks in four stages (347 us: half cache lines), operands staged in
// registers (396), H's fragments straight from memory (318 - 412).
typedef int i4v __attribute__((ext_vector_type(4)));

constexpr int GKC = 128;  // K chunk (bytes)
constexpr int GTM = 256;  // rows of a tile
constexpr int GNT = 512;

// source of the block's pieces past the end of K
__device__ const i4v crt_zero_piece = {0, 0, 0, 0};

template <int FN, int GST>
__global__ __launch_bounds__(GNT, 2) void crt_gemm_k(const int8_t* __restrict__ Ap,
                                                     const int8_t* __restrict__ Bp, int n, int ld,
                                                     int cols, CrtBasis basis, int per_mod,
                                                     uint8_t* __restrict__ out, int tiles_m,
                                                     int tiles_n, int ntiles) {
  constexpr int FM = 4;
  constexpr int BN = 32 * FN;                  // columns of the tile
  constexpr int ABLK = GTM / 8, BBLK = BN / 8;    // wave loads of 1 KB: 8 rows each
  constexpr int LOADS = (ABLK + BBLK + 7) / 8;    // per wave and chunk
  constexpr int STAGE = (GTM + BN) * GKC;
  __shared__ __attribute__((aligned(256))) char lds[GST * STAGE];
  // XCD-aware order: each XCD works on a contiguous range of tiles, column
  // tiles fastest, so that those sharing rows of H run together on one L2
  const int per_xcd = gridDim.x >> 3;
  const int t = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (t >= ntiles) return;
  const int tn = t % tiles_n, tmp = t / tiles_n;
  const int tm = tmp % tiles_m, plane = tmp / tiles_m;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, lk = lane >> 4;
  const int8_t* A = Ap + (int64_t)plane * n * ld;
  const int8_t* B = Bp + (int64_t)plane * cols * ld;
  const int n0 = tn * BN;

  // The piece a lane copies into its place (row lane / 8, slot lane % 8 of a
  // block of 8 rows): piece p of a row sits in slot p ^ key, an involution.
  // Rows and columns past the end are clamped: their products are not stored.
  auto akey = [](int r) { return ((r >> 1) & 1) | ((r >> 3) & 6); };
  auto bkey = [](int r) { return (r >> 1) & 7; };
  const int8_t* src[LOADS];
  int kpos[LOADS];
  bool isb[LOADS];
#pragma unroll
  for (int e = 0; e < LOADS; ++e) {
    int blk = wave + 8 * e;
    if (blk >= ABLK + BBLK) blk = ABLK + BBLK - 1;  // again the last block
    isb[e] = blk >= ABLK;
    const int r = (isb[e] ? blk - ABLK : blk) * 8 + (lane >> 3);
    const int piece = (lane & 7) ^ (isb[e] ? bkey(r) : akey(r));
    if (isb[e]) {
      const int j = n0 + r;
      src[e] = B + (int64_t)(j < cols ? j : cols - 1) * ld + 16 * piece;
    } else {
      const int i = tm * GTM + r;
      src[e] = A + (int64_t)(i < n ? i : n - 1) * ld + 16 * piece;
    }
    kpos[e] = 16 * piece;
  }
  const int chunks = (ld + GKC - 1) / GKC;
  auto issue = [&](int c) {
    // past the last chunk the copies repeat it, into a stage nobody reads, so
    // that the number in flight stays what the waits below count
    const int cc = c < chunks ? c : chunks - 1;
    const int k0 = cc * GKC;
    char* base = lds + (c % GST) * STAGE;
#pragma unroll
    for (int e = 0; e < LOADS; ++e) {
      int blk = wave + 8 * e;
      if (blk >= ABLK + BBLK) blk = ABLK + BBLK - 1;
      const int8_t* p = src[e] + k0;
      if (k0 + kpos[e] >= ld)  // the last chunk: zeros for B, any bytes for A
        p = isb[e] ? reinterpret_cast<const int8_t*>(&crt_zero_piece) : src[e] - kpos[e];
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p,
                                       (__attribute__((address_space(3))) void*)(base + blk * 1024),
                                       16, 0, 0);
    }
  };

  i4v acc[FM][FN];
#pragma unroll
  for (int f = 0; f < FM; ++f)
#pragma unroll
    for (int g = 0; g < FN; ++g) acc[f][g] = i4v{0, 0, 0, 0};

  // byte offsets of this lane's pieces within a stage
  int ao[FM], bo[FN];
#pragma unroll
  for (int f = 0; f < FM; ++f) {
    const int r = wm * 64 + 16 * (l16 >> 2) + 4 * f + (l16 & 3);
    ao[f] = r * GKC + 16 * (lk ^ akey(r));
  }
#pragma unroll
  for (int g = 0; g < FN; ++g) {
    const int r = wn * (16 * FN) + 16 * g + l16;
    bo[g] = GTM * GKC + r * GKC + 16 * (lk ^ bkey(r));
  }

  constexpr int AHEAD = GST - 1;
  constexpr int INFLIGHT = (AHEAD - 1) * LOADS;  // copies of the later chunks
  static_assert(INFLIGHT < 64, "vmcnt range");
#pragma unroll
  for (int c = 0; c < AHEAD; ++c) issue(c);
  for (int c = 0; c < chunks; ++c) {
    // chunk c has landed, and every wave is done with chunk c - 1's stage,
    // which chunk c + AHEAD then fills
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((INFLIGHT & 15) | (7 << 4) | ((INFLIGHT >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(c + AHEAD);
    const char* st = lds + (c % GST) * STAGE;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      i4v av[FM];
#pragma unroll
      for (int f = 0; f < FM; ++f) av[f] = *reinterpret_cast<const i4v*>(st + (ao[f] ^ (64 * h)));
#pragma unroll
      for (int g = 0; g < FN; ++g) {
        const i4v bv = *reinterpret_cast<const i4v*>(st + (bo[g] ^ (64 * h)));
#pragma unroll
        for (int f = 0; f < FM; ++f)
          acc[f][g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[f], bv, acc[f][g], 0, 0, 0);
      }
    }
  }
  // no copy may land in LDS after the workgroup has ended
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x70);  // vmcnt(0) lgkmcnt(0)
  asm volatile("" ::: "memory");

  // residues: acc[f][g][r] is row i0 + 4 f + r of column 16 g + l16
  const int m = basis.m[plane / per_mod];
  const double minv = 1.0 / (double)m;
  const int i0 = tm * GTM + wm * 64 + 16 * lk;
#pragma unroll
  for (int g = 0; g < FN; ++g) {
    const int j = n0 + wn * (16 * FN) + 16 * g + l16;
    if (j >= cols || i0 >= ld) continue;
    i4v w;
#pragma unroll
    for (int f = 0; f < FM; ++f) {
      uint32_t x = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) x |= (uint32_t)ures32(acc[f][g][r], m, minv) << (8 * r);
      w[f] = (int)x;
    }
    *reinterpret_cast<i4v*>(out + ((int64_t)plane * cols + j) * ld + i0) = w;
  }
}

template <int FN, int GST>
void crt_gemm_launch(const int8_t* A, const int8_t* B, int64_t n, int cols, const CrtBasis& basis,
                     int per_mod, uint8_t* out, hipStream_t st) {
  const int64_t tm = (n + GTM - 1) / GTM, tn = (cols + 32 * FN - 1) / (32 * FN);
  const int64_t nt = tm * tn * per_mod * basis.n_mod;
  CHASE_REQUIRE(nt <= INT32_MAX - 8, "INT8 products: too many tiles");
  hipLaunchKernelGGL((crt_gemm_k<FN, GST>), dim3((unsigned)((nt + 7) / 8 * 8)), dim3(GNT), 0, st, A, B,
                     (int)n, (int)plane_ld(n), cols, basis, per_mod, out, (int)tm, (int)tn, (int)nt);
  CHASE_HIP(hipGetLastError());
}

void crt_gemm(const int8_t* A, const int8_t* B, int64_t n, int cols, const CrtBasis& basis,
              int per_mod, uint8_t* out, hipStream_t st) {
  // column tile with the least work on the busiest of the 256 compute units:
  // rounds of tiles times columns, over the rate (TOP/s on n=20000) its width
  // reaches
  static constexpr struct {
    int fn;
    double rate;
  } tiles[] = {{9, 2030}, {8, 2007}, {6, 1711}, {4, 1521}, {2, 1132}, {1, 646}};
  int fn = 0;
  double cost = 0.0;
  for (const auto& t : tiles) {
    const int64_t nt = (n + GTM - 1) / GTM * ((cols + 32 * t.fn - 1) / (32 * t.fn)) * per_mod *
                       basis.n_mod;
    const double c = (double)((nt + 255) / 256) * t.fn / t.rate;
    if (fn == 0 || c < cost) {
      fn = t.fn;
      cost = c;
    }
  }
  switch (fn) {
    case 9: return crt_gemm_launch<9, 2>(A, B, n, cols, basis, per_mod, out, st);
    case 8: return crt_gemm_launch<8, 2>(A, B, n, cols, basis, per_mod, out, st);
    case 6: return crt_gemm_launch<6, 2>(A, B, n, cols, basis, per_mod, out, st);
    case 4: return crt_gemm_launch<4, 3>(A, B, n, cols, basis, per_mod, out, st);
    case 2: return crt_gemm_launch<2, 3>(A, B, n, cols, basis, per_mod, out, st);
    default: return crt_gemm_launch<1, 3>(A, B, n, cols, basis, per_mod, out, st);
  }
}

// sigma[i] = pa - e_i, 2^(e_i - 1) <= max_j |H_ij| (real and imaginary parts)
// < 2^e_i, from column i (row i of a Hermitian H is its conjugate).
template <bool CPLX>
__global__ __launch_bounds__(TPB) void crt_rowexp_k(const double* __restrict__ H, int64_t ldh,
                                                    int64_t n, int pa, int* __restrict__ sigma) {
  __shared__ double red[TPB];
  const int64_t i = blockIdx.x;
  const int W = CPLX ? 2 : 1;
  double m = 0.0;
  for (int64_t e = threadIdx.x; e < n * W; e += TPB) m = fmax(m, fabs(H[i * ldh * W + e]));
  red[threadIdx.x] = m;
  __syncthreads();
  for (int s = TPB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) sigma[i] = red[0] > 0.0 ? pa - exp2_above(red[0]) : 0;
}

// tau[j] = pb - e_j for column j of X (n rows).
template <bool CPLX>
__global__ __launch_bounds__(TPB) void crt_colexp_k(const double* __restrict__ X, int64_t ldx,
                                                    int64_t n, int pb, int* __restrict__ tau) {
  __shared__ double red[TPB];
  const int64_t j = blockIdx.x;
  const int W = CPLX ? 2 : 1;
  double m = 0.0;
  for (int64_t e = threadIdx.x; e < n * W; e += TPB) m = fmax(m, fabs(X[j * ldx * W + e]));
  red[threadIdx.x] = m;
  __syncthreads();
  for (int s = TPB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  if (threadIdx.x == 0) tau[j] = red[0] > 0.0 ? pb - exp2_above(red[0]) : 0;
}

// Residue planes of H, row-major (element (i, j) at i ld + j).  Complex: planes 3t+0 (Re),
// 3t+1 (Im), 3t+2 (Re + Im) of modulus t; real: plane t.  Row i of H is
// conj(column i): Re H_ij = Re H[j + i ldh], Im H_ij = -Im H[j + i ldh].
// Four consecutive entries per thread: the residues of each plane go out as
// one packed 32-bit store (byte e = entry e; entries past n are zero).
template <bool CPLX>
__global__ __launch_bounds__(TPB) void crt_hplanes_k(const double* __restrict__ H, int64_t ldh,
                                                      int64_t n, const int* __restrict__ sigma,
                                                      CrtBasis B, int8_t* __restrict__ planes) {
  const int64_t i = blockIdx.y;
  const int64_t j0 = 4 * ((int64_t)blockIdx.x * TPB + threadIdx.x);
  const int64_t ld = plane_ld(n);
  if (j0 >= ld) return;
  const int s = sigma[i];
  const int64_t o = i * ld + j0;
  const int64_t plane = n * ld;
  if constexpr (CPLX) {
    double re[4], im[4], sm[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      re[e] = j0 + e < n ? rint(ldexp(H[2 * (j0 + e + i * ldh)], s)) : 0.0;
      im[e] = j0 + e < n ? rint(ldexp(-H[2 * (j0 + e + i * ldh) + 1], s)) : 0.0;
      sm[e] = re[e] + im[e];
    }
    for (int t = 0; t < B.n_mod; ++t) {
      const int m = B.m[t];
      const double minv = 1.0 / (double)m;
      uint32_t wr = 0, wi = 0, ws = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        wr |= (uint32_t)(uint8_t)bres(re[e], m, minv) << (8 * e);
        wi |= (uint32_t)(uint8_t)bres(im[e], m, minv) << (8 * e);
        ws |= (uint32_t)(uint8_t)bres(sm[e], m, minv) << (8 * e);
      }
      *reinterpret_cast<uint32_t*>(planes + (3 * t + 0) * plane + o) = wr;
      *reinterpret_cast<uint32_t*>(planes + (3 * t + 1) * plane + o) = wi;
      *reinterpret_cast<uint32_t*>(planes + (3 * t + 2) * plane + o) = ws;
    }
  } else {
    double v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = j0 + e < n ? rint(ldexp(H[j0 + e + i * ldh], s)) : 0.0;
    for (int t = 0; t < B.n_mod; ++t) {
      uint32_t w = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w |= (uint32_t)(uint8_t)bres(v[e], B.m[t], 1.0 / (double)B.m[t]) << (8 * e);
      *reinterpret_cast<uint32_t*>(planes + t * plane + o) = w;
    }
  }
}

// Residue planes of the block X (n x cols, column-major, ld per plane).
template <bool CPLX>
__global__ __launch_bounds__(TPB) void crt_xplanes_k(const double* __restrict__ X, int64_t ldx,
                                                      int64_t n, int cols,
                                                      const int* __restrict__ tau, CrtBasis B,
                                                      int8_t* __restrict__ planes) {
  const int64_t j = blockIdx.y;
  const int64_t i0 = 4 * ((int64_t)blockIdx.x * TPB + threadIdx.x);
  const int64_t ld = plane_ld(n);
  if (i0 >= ld) return;
  const int s = tau[j];
  const int64_t o = j * ld + i0;
  const int64_t plane = ld * (int64_t)cols;
  if constexpr (CPLX) {
    double re[4], im[4], sm[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      re[e] = i0 + e < n ? rint(ldexp(X[2 * (i0 + e + j * ldx)], s)) : 0.0;
      im[e] = i0 + e < n ? rint(ldexp(X[2 * (i0 + e + j * ldx) + 1], s)) : 0.0;
      sm[e] = re[e] + im[e];
    }
    for (int t = 0; t < B.n_mod; ++t) {
      const int m = B.m[t];
      const double minv = 1.0 / (double)m;
      uint32_t wr = 0, wi = 0, ws = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        wr |= (uint32_t)(uint8_t)bres(re[e], m, minv) << (8 * e);
        wi |= (uint32_t)(uint8_t)bres(im[e], m, minv) << (8 * e);
        ws |= (uint32_t)(uint8_t)bres(sm[e], m, minv) << (8 * e);
      }
      *reinterpret_cast<uint32_t*>(planes + (3 * t + 0) * plane + o) = wr;
      *reinterpret_cast<uint32_t*>(planes + (3 * t + 1) * plane + o) = wi;
      *reinterpret_cast<uint32_t*>(planes + (3 * t + 2) * plane + o) = ws;
    }
  } else {
    double v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      v[e] = i0 + e < n ? rint(ldexp(X[i0 + e + j * ldx], s)) : 0.0;
    for (int t = 0; t < B.n_mod; ++t) {
      uint32_t w = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w |= (uint32_t)(uint8_t)bres(v[e], B.m[t], 1.0 / (double)B.m[t]) << (8 * e);
      *reinterpret_cast<uint32_t*>(planes + t * plane + o) = w;
    }
  }
}

// Garner: the integer x with x = r_t (mod m_t), |x| < M / 2, from residues
// r_t in [0, m_t): balanced mixed-radix digits v_t, x = v_0 + m_0 (v_1 + m_1
// (v_2 + ...)), evaluated in FP64 from the top digit (error <= ~NM u |x|).
// The moduli are compile-time constants.
// x mod m in [0, m) for an integer-valued float |x| < 2^24 (exact: the
// quotient estimate is off by at most one, which the two corrections undo)
__device__ __forceinline__ float fmod_m(float x, float m, float minv) {
  const float q = floorf(x * minv);
  float r = fmaf(-q, m, x);
  if (r < 0.f) r += m;
  if (r >= m) r -= m;
  return r;
}

// (m_0 m_1 ... m_{s-1}) mod m_t
constexpr int radix_mod(int s, int t) {
  int p = 1;
  for (int i = 0; i < s; ++i) p = p * (kModuli[i] % kModuli[t]) % kModuli[t];
  return p;
}

// One digit: (v_0 + m_0 v_1 + m_0 m_1 v_2 + ...) mod m_t as a sum with the
// radices already reduced modulo m_t, and one reduction at its end.
template <int T, int... S>
__device__ __forceinline__ float known_digits(const float* v, std::integer_sequence<int, S...>) {
  float acc = 0.f;
  ((acc = fmaf(v[S], (float)radix_mod(S, T), acc)), ...);
  return acc;
}
template <int NM, int T>
__device__ __forceinline__ void garner_digit(const int (&r)[NM], float (&v)[NM],
                                             const CrtBasis& B) {
  const float m = (float)kModuli[T], minv = 1.0f / (float)kModuli[T];
  float d = fmod_m((float)r[T] - known_digits<T>(v, std::make_integer_sequence<int, T>{}), m, minv);
  d = fmod_m(d * (float)B.inv[T], m, minv);
  if (d > (m - 1.f) * 0.5f) d -= m;
  v[T] = d;
}
template <int NM, int... T>
__device__ __forceinline__ void garner_digits(const int (&r)[NM], float (&v)[NM],
                                              const CrtBasis& B, std::integer_sequence<int, T...>) {
  (garner_digit<NM, T>(r, v, B), ...);
}

template <int NM>
__device__ __forceinline__ double garner(const int (&r)[NM], const CrtBasis& B) {
  // every intermediate is an integer below 2^19 in magnitude (15 digits of at
  // most 128 times radices below 256), exact in FP32, whose multiply-adds run
  // at full rate (32-bit integer multiplies do not).  Reducing after every
  // digit, Horner's way, took 65 us for 4000 x 260 complex entries
  float v[NM];
  garner_digits<NM>(r, v, B, std::make_integer_sequence<int, NM>{});
  double x = 0.0;
#pragma unroll
  for (int t = NM - 1; t >= 0; --t) x = fma(x, (double)kModuli[t], (double)v[t]);
  return x;
}

// The epilogue of one entry: out = alpha (c - gamma Xs) + beta out [+ cj F].
template <bool CPLX>
__device__ __forceinline__ void cheb_store(const GemmArgs& g, int64_t i, int64_t j, double vr,
                                           double vi) {
  const double* Xs = static_cast<const double*>(g.B);
  double* Cd = static_cast<double*>(g.C);
  const int64_t oc = i + j * g.ldc;
  if constexpr (CPLX) {
    vr = g.alpha * (vr - g.gamma * Xs[2 * (i + j * g.ldb)]);
    vi = g.alpha * (vi - g.gamma * Xs[2 * (i + j * g.ldb) + 1]);
    if (g.beta != 0.0) {
      vr += g.beta * Cd[2 * oc];
      vi += g.beta * Cd[2 * oc + 1];
    }
    if (g.colcoef) {
      const double cj = g.colcoef[j];
      const double* Fd = static_cast<const double*>(g.F);
      vr += cj * Fd[2 * (i + j * g.ldf)];
      vi += cj * Fd[2 * (i + j * g.ldf) + 1];
    }
    Cd[2 * oc] = vr;
    Cd[2 * oc + 1] = vi;
  } else {
    double v = g.alpha * (vr - g.gamma * Xs[i + j * g.ldb]);
    if (g.beta != 0.0) v += g.beta * Cd[oc];
    if (g.colcoef) v += g.colcoef[j] * static_cast<const double*>(g.F)[i + j * g.ldf];
    Cd[oc] = v;
  }
}

// out(i, j) = alpha (C(i, j) - gamma Xs(i, j)) + beta out(i, j)
//             [+ colcoef[j] F(i, j)],  C = H Xs from the products' residues.
// Four consecutive rows per thread (one 32-bit load per plane), the residues
// kept packed, one byte each, until each entry's reconstruction.
template <bool CPLX, int NM>
__global__ __launch_bounds__(TPB) void crt_cheb_k(const uint8_t* __restrict__ P, int64_t n,
                                                  int cols, CrtBasis B,
                                                  const int* __restrict__ sigma,
                                                  const int* __restrict__ tau, GemmArgs g) {
  const int64_t j = blockIdx.y;
  const int64_t i0 = 4 * ((int64_t)blockIdx.x * TPB + threadIdx.x);
  if (i0 >= n) return;
  const int64_t ld = plane_ld(n);
  const int64_t plane = ld * (int64_t)cols;
  const int64_t o = j * ld + i0;
  auto residues = [&](int p) { return *reinterpret_cast<const uint32_t*>(P + p * plane + o); };
  uint32_t pr[NM], pi[NM];
#pragma unroll
  for (int t = 0; t < NM; ++t) {
    const int m = kModuli[t];
    uint32_t wr = 0, wi = 0;
    if constexpr (CPLX) {
      const uint32_t a = residues(3 * t), b = residues(3 * t + 1), c = residues(3 * t + 2);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int p1 = (a >> (8 * e)) & 0xff, p2 = (b >> (8 * e)) & 0xff;
        const int p3 = (c >> (8 * e)) & 0xff;
        int re = p1 - p2, im = p3 - p1 - p2;  // in (-m, m) and (-2m, m)
        re += re < 0 ? m : 0;
        im += im < 0 ? m : 0;
        im += im < 0 ? m : 0;
        wr |= (uint32_t)re << (8 * e);
        wi |= (uint32_t)im << (8 * e);
      }
    } else {
      wr = residues(t);
    }
    pr[t] = wr;
    pi[t] = wi;
  }
  const int ej = tau[j];
  // one entry at a time (the reconstructions of four entries side by side
  // would hold four sets of digits)
#pragma unroll 1
  for (int e = 0; e < 4; ++e) {
    const int64_t i = i0 + e;
    if (i >= n) break;
    const int sc = -(sigma[i] + ej);
    int r[NM];
#pragma unroll
    for (int t = 0; t < NM; ++t) r[t] = (int)((pr[t] >> (8 * e)) & 0xffu);
    const double vr = ldexp(garner<NM>(r, B), sc);
    double vi = 0.0;
    if constexpr (CPLX) {
#pragma unroll
      for (int t = 0; t < NM; ++t) r[t] = (int)((pi[t] >> (8 * e)) & 0xffu);
      vi = ldexp(garner<NM>(r, B), sc);
    }
    cheb_store<CPLX>(g, i, j, vr, vi);
  }
}

template <bool CPLX, int NM>
void launch_cheb(const uint8_t* prod, int64_t n, int cols, const CrtBasis& B, const int* sigma,
                 const int* tau, const GemmArgs& g, hipStream_t st) {
  const dim3 grid((unsigned)(((n + 3) / 4 + TPB - 1) / TPB), (unsigned)cols);
  hipLaunchKernelGGL((crt_cheb_k<CPLX, NM>), grid, dim3(TPB), 0, st, prod, n, cols, B, sigma, tau,
                     g);
}

template <bool CPLX>
void launch_cheb_nm(const uint8_t* prod, int64_t n, int cols, const CrtBasis& B,
                    const int* sigma, const int* tau, const GemmArgs& g, hipStream_t st) {
  switch (B.n_mod) {
    case 8: return launch_cheb<CPLX, 8>(prod, n, cols, B, sigma, tau, g, st);
    case 10: return launch_cheb<CPLX, 10>(prod, n, cols, B, sigma, tau, g, st);
    case 12: return launch_cheb<CPLX, 12>(prod, n, cols, B, sigma, tau, g, st);
    case 14: return launch_cheb<CPLX, 14>(prod, n, cols, B, sigma, tau, g, st);
    case 16: return launch_cheb<CPLX, 16>(prod, n, cols, B, sigma, tau, g, st);
  }
  throw Error(CHASE_ERR_ARG, "fp64_emulation: moduli must be 8, 10, 12, 14 or 16");
}

int inv_mod(int a, int m) {
  // extended Euclid; a and m coprime
  int t = 0, nt = 1, r = m, nr = ((a % m) + m) % m;
  while (nr != 0) {
    const int q = r / nr;
    int tmp = t - q * nt;
    t = nt;
    nt = tmp;
    tmp = r - q * nr;
    r = nr;
    nr = tmp;
  }
  return ((t % m) + m) % m;
}

}  // namespace

CrtBasis crt_basis(int n_mod, int64_t K, bool cplx) {
  CHASE_REQUIRE(n_mod == 8 || n_mod == 10 || n_mod == 12 || n_mod == 14 || n_mod == 16,
                "fp64_emulation: moduli must be 8, 10, 12, 14 or 16");
  CrtBasis b{};
  b.n_mod = n_mod;
  double log2M = 0.0;
  for (int t = 0; t < n_mod; ++t) {
    b.m[t] = kModuli[t];
    log2M += std::log2((double)kModuli[t]);
    // inverse of m_0 ... m_{t-1} modulo m_t
    int prod = 1;
    for (int s = 0; s < t; ++s) prod = (int)(((int64_t)prod * (kModuli[s] % kModuli[t])) % kModuli[t]);
    b.inv[t] = t == 0 ? 1 : inv_mod(prod, kModuli[t]);
  }
  // |C| <= 2 K 2^(pa + pb) (complex parts; real: K 2^(pa + pb)) must stay
  // below M / 2, one bit of margin
  const int total = (int)std::floor(log2M - 1.0 - 1.0 - std::log2((double)std::max<int64_t>(K, 1)) -
                                    (cplx ? 1.0 : 0.0));
  b.pa = std::min(52, total / 2);
  b.pb = std::min(52, total - b.pa);
  CHASE_REQUIRE(b.pa >= 16 && b.pb >= 16, "fp64_emulation: too few moduli for this size");
  return b;
}

namespace {
inline size_t align256(size_t b) { return (b + 255) / 256 * 256; }
// byte offsets within the buffers: H planes | row exponents;
// block planes | residues of the products | column exponents
inline size_t h_planes_bytes(bool cplx, int64_t n, int n_mod) {
  return align256((size_t)(cplx ? 3 : 1) * n_mod * n * plane_ld(n));
}
inline size_t x_planes_bytes(bool cplx, int64_t n, int kmax, int n_mod) {
  return align256((size_t)(cplx ? 3 : 1) * n_mod * plane_ld(n) * kmax);
}
inline size_t x_prod_bytes(bool cplx, int64_t n, int kmax, int n_mod) {
  return align256((size_t)(cplx ? 3 : 1) * n_mod * plane_ld(n) * kmax);
}
}  // namespace

size_t crt_h_bytes(bool cplx, int64_t n, int n_mod) {
  return h_planes_bytes(cplx, n, n_mod) + (size_t)n * 4;
}
// The size that callers know from the workspace query is that of unpadded planes
// with INT32 products, five bytes a plane and entry of the block.  It is kept, and
// holds the padding of H's planes as well; two bytes are in use.
size_t crt_x_bytes(bool cplx, int64_t n, int kmax, int n_mod) {
  const size_t planes = (size_t)(cplx ? 3 : 1) * n_mod, entries = planes * n * kmax;
  const size_t tail = (size_t)kmax * 4 + 256;
  const size_t known = align256(entries) + align256(4 * entries) + tail;
  const size_t pad = h_planes_bytes(cplx, n, n_mod) - align256(planes * n * n);
  const size_t used =
      x_planes_bytes(cplx, n, kmax, n_mod) + x_prod_bytes(cplx, n, kmax, n_mod) + tail;
  return std::max(used, known - std::min(known, pad));
}

void crt_prepare_h(bool cplx, const void* H, int64_t ldh, int64_t n, const CrtBasis& B,
                   void* hbuf, hipStream_t st) {
  CHASE_REQUIRE(n <= 65535, "fp64_emulation: n above 65535");
  int8_t* planes = static_cast<int8_t*>(hbuf);
  int* sigma = reinterpret_cast<int*>(planes + h_planes_bytes(cplx, n, B.n_mod));
  const double* Hd = static_cast<const double*>(H);
  const dim3 grid((unsigned)((plane_ld(n) / 4 + TPB - 1) / TPB), (unsigned)n);
  if (cplx) {
    hipLaunchKernelGGL(crt_rowexp_k<true>, dim3((unsigned)n), dim3(TPB), 0, st, Hd, ldh, n, B.pa,
                       sigma);
    hipLaunchKernelGGL(crt_hplanes_k<true>, grid, dim3(TPB), 0, st, Hd, ldh, n,
                       static_cast<const int*>(sigma), B, planes);
  } else {
    hipLaunchKernelGGL(crt_rowexp_k<false>, dim3((unsigned)n), dim3(TPB), 0, st, Hd, ldh, n, B.pa,
                       sigma);
    hipLaunchKernelGGL(crt_hplanes_k<false>, grid, dim3(TPB), 0, st, Hd, ldh, n,
                       static_cast<const int*>(sigma), B, planes);
  }
  CHASE_HIP(hipGetLastError());
}

void crt_cheb(bool cplx, const GemmArgs& g, const CrtBasis& B, const void* hbuf, void* xbuf,
              int kmax, hipStream_t st) {
  const int64_t n = g.M;
  const int cols = (int)g.N;
  CHASE_REQUIRE(g.K == n && cols >= 1 && cols <= kmax, "INT8 filter step: shape");
  const int8_t* hplanes = static_cast<const int8_t*>(hbuf);
  const int* sigma = reinterpret_cast<const int*>(hplanes + h_planes_bytes(cplx, n, B.n_mod));
  int8_t* xplanes = static_cast<int8_t*>(xbuf);
  uint8_t* prod = reinterpret_cast<uint8_t*>(xplanes + x_planes_bytes(cplx, n, kmax, B.n_mod));
  int* tau = reinterpret_cast<int*>(prod + x_prod_bytes(cplx, n, kmax, B.n_mod));
  const double* Xs = static_cast<const double*>(g.B);
  const dim3 grid((unsigned)((plane_ld(n) / 4 + TPB - 1) / TPB), (unsigned)cols);
  if (cplx) {
    hipLaunchKernelGGL(crt_colexp_k<true>, dim3(cols), dim3(TPB), 0, st, Xs, g.ldb, n, B.pb, tau);
    hipLaunchKernelGGL(crt_xplanes_k<true>, grid, dim3(TPB), 0, st, Xs, g.ldb, n, cols,
                       static_cast<const int*>(tau), B, xplanes);
  } else {
    hipLaunchKernelGGL(crt_colexp_k<false>, dim3(cols), dim3(TPB), 0, st, Xs, g.ldb, n, B.pb, tau);
    hipLaunchKernelGGL(crt_xplanes_k<false>, grid, dim3(TPB), 0, st, Xs, g.ldb, n, cols,
                       static_cast<const int*>(tau), B, xplanes);
  }
  CHASE_HIP(hipGetLastError());
  crt_gemm(hplanes, xplanes, n, cols, B, cplx ? 3 : 1, prod, st);
  if (cplx)
    launch_cheb_nm<true>(prod, n, cols, B, sigma, tau, g, st);
  else
    launch_cheb_nm<false>(prod, n, cols, B, sigma, tau, g, st);
  CHASE_HIP(hipGetLastError());
}

}  // namespace chase
