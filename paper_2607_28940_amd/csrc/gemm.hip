// Projection and FFN GEMMs of the TransX path: C = epi(A * Bt^T + bias [+ R]).
//
// A is the packed activation matrix [M][K] (token rows), Bt the repacked weight
// [N][K] (the layer's W [K][N] transposed so that both operands are contiguous
// along K). Epilogues: +bias, +bias then exact-erf GELU (FFN), +bias + residual
// (post-LN sublayers add the block input before LayerNorm, Sec. 4.1.2). A
// residual that is itself a LayerNorm output is recomputed in fp32 from the
// stored pre-LN sum and its row statistics, so the residual stream never
// passes through the rounded bf16 copy the sublayer used as its operand, and
// the new pre-LN sum is stored in fp16 (see EPI_BIAS_RESLN).
//
// bf16 path: v_mfma_f32_32x32x16_bf16 with fp32 accumulation. The weight tile
// is the MFMA "A" operand and the activation tile the "B" operand, so each
// lane's accumulator holds 4 consecutive output columns of one row. Large
// products run on a persistent kernel (one block per CU walking 256x256 tiles,
// see gemm_bf16_p4); the others on one block per tile of 32x32 to 128x128
// (gemm_bf16_ring) or of 128x128 with two blocks per CU (gemm_bf16_pair), by
// estimated time (gemm_plan.h). Tiles are numbered so that each of the 8 XCDs
// (the hardware deals workgroup b to XCD b % 8) works through a contiguous
// range of them, walked in groups of row blocks so that operand
// blocks are reused from that XCD's L2.
#include <atomic>

#include "gemm_plan.h"
#include "tx_internal.h"

#include <algorithm>
#include <type_traits>

namespace tx {

// GELU(x) = x Phi(x) = max(x, 0) - u Phi(-u) with u = |x|, for either sign
// of x. Phi(-u) = 2^Q(min(u, 6)) with Q a degree-7 least-squares fit to
// log2 Phi(-u) on Chebyshev nodes of [0, 6] (gelu_fit.py): fractional error
// below 5.5e-6 for |x| <= 6 (evaluated in fp32), 360 times below the bf16
// output's half unit; beyond, where |GELU(x)| < 1e-9 |x|, the clamp keeps the
// error below that. Seven FMAs, one exp2 and no reciprocal.
__device__ __forceinline__ float gelu_erf(float x) {
  const float u = fminf(fabsf(x), 6.0f);
  float q = -1.889626233332388e-06f;
  q = fmaf(q, u, 6.268140100811885e-05f);
  q = fmaf(q, u, -0.0009388679332881356f);
  q = fmaf(q, u, 0.008539461331933599f);
  q = fmaf(q, u, -0.05402068711617134f);
  q = fmaf(q, u, -0.45840977680772027f);
  q = fmaf(q, u, -1.1512691471649812f);
  q = fmaf(q, u, -0.9999943403320692f);
  return fmaf(-fabsf(x), __builtin_amdgcn_exp2f(q), fmaxf(x, 0.f));
}

template <int EPI>
__device__ __forceinline__ float epilogue(float acc, float bias, float resid) {
#pragma clang fp contract(off)
  float v = acc + bias;
  if (epi_gelu(EPI)) v = gelu_erf(v);
  if (epi_resid(EPI)) v += resid;
  return v;
}

// Residual element e of a 16-byte piece of R: the model-type value itself
// (EPI_BIAS_RESID) or the LayerNorm of the fp16 pre-LN sum with row
// statistics st and the column's gain g (EPI_BIAS_RESLN), whose offset every
// kernel adds to the bias instead: (acc + (bias + b)) + (y * x + y') * g, the
// same operations in the same order in each kernel, so that they agree
// bitwise.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float ln_resid(float y, LnRow st, float g) {
#pragma clang fp contract(off)
  return fmaf(y, st.x, st.y) * g;
}
template <int EPI>
__device__ __forceinline__ float resid8(const u32x4& raw, int e, LnRow st, float g) {
  if (EPI == EPI_BIAS_RESID) return (float)__builtin_bit_cast(bf16x8, raw)[e];
  if (EPI == EPI_BIAS_RESLN) return ln_resid((float)__builtin_bit_cast(f16x8, raw)[e], st, g);
  return 0.f;
}
template <int EPI>
__device__ __forceinline__ float resid4(const u32x2& raw, int e, LnRow st, float g) {
  if (EPI == EPI_BIAS_RESID) return (float)__builtin_bit_cast(bf16x4, raw)[e];
  if (EPI == EPI_BIAS_RESLN) return ln_resid((float)__builtin_bit_cast(f16x4, raw)[e], st, g);
  return 0.f;
}

// Epilogue and stores of one 32x32 accumulator: element v is column
// nb + 8 (v / 4) + v % 4 of row m (the lane's hi half already in nb); rrow is
// the residual's row (the model or the sum type, both 16 bits wide).
template <int EPI>
__device__ __forceinline__ void store_acc(const floatx16& acc, int m, int nb, const float* __restrict__ bias,
                                          const bf16* __restrict__ rrow, void* __restrict__ C, int ldc,
                                          const LnResid& ln) {
  LnRow st{0.f, 0.f};
  if (EPI == EPI_BIAS_RESLN || epi_lnfold(EPI)) st = ln.stats[m];
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int n = nb + 8 * g;
    floatx4 b4 = *reinterpret_cast<const floatx4*>(bias + n);
    if (epi_lnfold(EPI)) {
      // the same operations as the persistent kernel's epilogue
      const floatx4 cs4 = *reinterpret_cast<const floatx4*>(ln.g + n);
      bf16x4 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float v = fmaf(acc[4 * g + q], st.x, fmaf(st.y, cs4[q], b4[q]));
        if (epi_gelu(EPI)) v = gelu_erf(v);
        o[q] = (bf16)v;
      }
      *reinterpret_cast<bf16x4*>((bf16*)C + (size_t)m * ldc + n) = o;
    } else if (epi_resid(EPI)) {
      const u32x2 raw = *reinterpret_cast<const u32x2*>(rrow + n);
      floatx4 g4 = {0.f, 0.f, 0.f, 0.f};
      if (EPI == EPI_BIAS_RESLN) {
        g4 = *reinterpret_cast<const floatx4*>(ln.g + n);
        b4 += *reinterpret_cast<const floatx4*>(ln.b + n);
      }
      f16x4 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = (f16)epilogue<EPI>(acc[4 * g + q], b4[q], resid4<EPI>(raw, q, st, g4[q]));
      *reinterpret_cast<f16x4*>((f16*)C + (size_t)m * ldc + n) = o;
    } else {
      bf16x4 o;
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = (bf16)epilogue<EPI>(acc[4 * g + q], b4[q], 0.f);
      *reinterpret_cast<bf16x4*>((bf16*)C + (size_t)m * ldc + n) = o;
    }
  }
}

// s_waitcnt vmcnt(N) (loads of this wave except the N youngest have landed) and lgkmcnt(0), then the block's barrier.
template <int N>
struct RingWait {
  static __device__ __forceinline__ void go() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));  // vmcnt(N) lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
};
template <int S, int I = 0, class F>
__device__ __forceinline__ void ring_tail(F f) {
  f(std::integral_constant<int, I>{});
  if constexpr (I + 1 < S) ring_tail<S, I + 1>(f);
}

constexpr int RK = kRingK;  // k columns per stage

// Ring kernel: one block of four waves per BM x BN output tile, for products
// with too few 256x256 tiles for the persistent kernel. What bounds a small
// product is the latency of its operand loads and the serial chain of a
// block's k steps, so the operands travel HBM/L2 -> LDS with
// buffer_load_dwordx4 ... lds (no registers) through a ring of S stages of 64
// k columns, S requested ahead, and each k step costs one barrier: stage k + 1
// has landed (a counted vmcnt) and every wave has read stage k's fragments,
// so stage k's buffer takes the loads of stage k + S while the fragments of
// stage k + 1 are read between the MFMAs of stage k. Rows are 128 bytes, 16-byte
// slot s of row r holding chunk s ^ ((r / 2) % 8) (applied on the global
// side): conflict-free fragment reads without padding. A wave computes
// MI x NI MFMA tiles. The 32x32 and 32x64 tiles hold work for one or two waves;
// the others load their share and repeat those waves' products, which are
// dropped (leaving them out of the compute instead: one user's call 97.6 us
// either way, a session 442 against 438). Each output is summed over k in the same order
// with the same MFMAs as in the persistent kernel, so a score does not depend
// on which kernel took its batch. Measured per launch, against the pair kernel
// (128x128 tiles, operands through registers, one step ahead): M 34,
// N 512, K 2048 26 -> 6.3 us; M 34, N 1024, K 4096 48 -> 9.5; M 300 51 -> 12;
// M 1064 52 -> 21; M 4000 55 -> 37; M 1064, N 3072, K 1024 17.5 -> 11.3.
template <int EPI, int BM, int BN, int MI, int NI, int S>
__global__ __launch_bounds__(256) void gemm_bf16_ring(const bf16* __restrict__ A, int lda, const bf16* __restrict__ Bt,
                                                      const float* __restrict__ bias, const void* __restrict__ R,
                                                      int ldr, void* __restrict__ C, int ldc, int M, int N, int K,
                                                      int tiles_m1, int tiles_m, int tiles_n, bool n_major,
                                                      LnResid ln) {
  constexpr int ROWS = BM + BN, LPW = ROWS / 32;  // 1 KB loads per wave and stage
  constexpr int CWM = BM / (32 * MI), CW = CWM * (BN / (32 * NI));  // waves that compute
  static_assert(CW >= 1 && CW <= 4 && S >= 4 && S % 2 == 0 && ROWS % 32 == 0, "tile shape");
  __shared__ __attribute__((aligned(16))) bf16 lds[S * ROWS * RK];
  typedef __attribute__((address_space(3))) void* lds_ptr_t;

  const int n_tiles = tiles_m * tiles_n, per_xcd = (n_tiles + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (t >= n_tiles) return;
  const int mt = n_major ? t % tiles_m : t / tiles_n, nt = n_major ? t / tiles_m : t % tiles_n;
  // row tiles from tiles_m1 on lie in the second array (see LnResid::a2)
  const bool second = mt >= tiles_m1;
  const int row0 = second ? ln.m1 : 0;                            // output row of the array's row 0
  const int rows = second ? M - ln.m1 : (ln.a2 ? ln.m1 : M);      // rows of the array
  const int m0 = (second ? mt - tiles_m1 : mt) * BM, n0 = nt * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi = lane >> 5;

  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      second ? (void*)ln.a2 : (void*)A, 0, (int)(2u * (uint32_t)rows * (uint32_t)lda), 0x00020000);
  const __amdgpu_buffer_rsrc_t rb =
      __builtin_amdgcn_make_buffer_rsrc((void*)Bt, 0, (int)(2u * (uint32_t)N * (uint32_t)K), 0x00020000);
  // Load u of a wave fills rows 32 u + 8 wave .. + 7 of the stage (A rows, then
  // B rows): one byte offset per load, k0 in the scalar offset. Rows past M
  // lie beyond the A resource; their results are not stored.
  uint32_t off[LPW];
#pragma unroll
  for (int u = 0; u < LPW; ++u) {
    const int r = 32 * u + 8 * wave + (lane >> 3);
    const int c = ((lane & 7) ^ ((r >> 1) & 7)) * 16;
    off[u] = 32 * u < BM ? 2u * (uint32_t)(m0 + r) * (uint32_t)lda + c : 2u * (uint32_t)(n0 + r - BM) * (uint32_t)K + c;
  }
  const int nk = K / RK;
  constexpr int STAGE = ROWS * RK * 2;  // bytes
  int wr = 0, rd = 0;  // ring positions (byte offsets) of the next stage requested and the next read
  auto issue = [&](int kt) {
    bf16* dst = (bf16*)((char*)lds + wr) + wave * 512;
    wr = wr == (S - 1) * STAGE ? 0 : wr + STAGE;
#pragma unroll
    for (int u = 0; u < LPW; ++u)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(32 * u < BM ? ra : rb, (lds_ptr_t)(dst + 2048 * u), 16, (int)off[u],
                                               kt * (2 * RK), 0, 0);
  };
  const int wm = (wave % CW) % CWM, wn = (wave % CW) / CWM;
  floatx16 acc[NI][MI];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < MI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  struct Frags {
    bf16x8 a[4][MI], b[4][NI];
  };
  int fo[4];  // byte offsets of the lane's fragments of a stage, per 16-wide k sub-step
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) fo[ks] = l32 * 128 + (((2 * ks + hi) ^ ((l32 >> 1) & 7)) << 4);
  const int wa = wm * MI * 4096, wb = BM * 128 + wn * NI * 4096;
  auto fread = [&](Frags& f) {
    const int base = rd;
    rd = rd == (S - 1) * STAGE ? 0 : rd + STAGE;
    const char* sa = (const char*)lds + (base + wa);
    const char* sb = (const char*)lds + (base + wb);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
#pragma unroll
      for (int j = 0; j < MI; ++j) f.a[ks][j] = *reinterpret_cast<const bf16x8*>(sa + fo[ks] + j * 4096);
#pragma unroll
      for (int i = 0; i < NI; ++i) f.b[ks][i] = *reinterpret_cast<const bf16x8*>(sb + fo[ks] + i * 4096);
    }
  };
  auto mfma = [&](const Frags& f) {
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j) {
          if (epi_lnfold(EPI))
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, f.b[ks][i]),
                                                               __builtin_bit_cast(f16x8, f.a[ks][j]), acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[ks][i], f.a[ks][j], acc[i][j], 0, 0, 0);
        }
  };
  // a stage's MFMAs, the next stage's fragment reads between the first half of
  // them (so that they have landed by the barrier) and D loads between the others
  auto pace = [&](auto D_) {
    constexpr int ND = decltype(D_)::value, NM = 4 * MI * NI, NR = 4 * (MI + NI), H = NM / 2;
#pragma unroll
    for (int g = 0; g < NM; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (g < H) __builtin_amdgcn_sched_group_barrier(0x100, NR / H, 0);
      else if (ND) __builtin_amdgcn_sched_group_barrier(0x020, (ND + NM - H - 1) / (NM - H), 0);
    }
  };
  auto next = [&](Frags& cur, Frags& nxt) {
    fread(nxt);
    mfma(cur);
    pace(std::integral_constant<int, 0>{});
  };
  const int pre = min(S, nk);
  for (int s = 0; s < pre; ++s) issue(s);
  // stage 0: the loads of stages 1 .. pre - 1 may stay in flight
  if (pre == S) RingWait<(S - 1) * LPW>::go();
  else if (pre == S / 2) RingWait<(S / 2 - 1) * LPW>::go();
  else RingWait<0>::go();
  Frags f0, f1;  // stage kt's fragments are in f0 when nk - kt is even
  if (nk & 1) fread(f1);
  else fread(f0);
  int kt = 0;
  auto steady = [&](Frags& cur, Frags& nxt) {
    RingWait<(S - 2) * LPW>::go();  // stage kt + 1 landed, stage kt's fragments read by every wave
    fread(nxt);
    issue(kt + S);
    mfma(cur);
    pace(std::integral_constant<int, LPW>{});
    ++kt;
  };
  if (nk > S && (nk & 1)) steady(f1, f0);
  while (kt + S < nk) {
    steady(f0, f1);
    steady(f1, f0);
  }
  // the last S stages: nothing left to request
  ring_tail<S>([&](auto I_) {
    constexpr int I = decltype(I_)::value;  // S - I stages left, this one included
    if (S - I > nk) return;
    RingWait<(I < S - 1 ? S - 2 - I : 0) * LPW>::go();
    Frags& cur = (S - I) & 1 ? f1 : f0;
    Frags& nxt = (S - I) & 1 ? f0 : f1;
    if (I < S - 1) next(cur, nxt);
    else mfma(cur);
  });
  if (wave >= CW) return;
#pragma unroll
  for (int j = 0; j < MI; ++j) {
    const int m = m0 + (wm * MI + j) * 32 + l32;
    if (m >= rows) continue;
    const bf16* rrow = (const bf16*)(second ? ln.r2 : R) + (size_t)m * ldr;
#pragma unroll
    for (int i = 0; i < NI; ++i)
      store_acc<EPI>(acc[i][j], row0 + m, n0 + (wn * NI + i) * 32 + 4 * hi, bias, rrow, C, ldc, ln);
  }
}

// Pair kernel: one block of four waves per 128x128 output tile, two blocks per
// CU, operands staged global -> registers -> LDS (rows padded by 16 bytes, no
// bank conflicts), double-buffered, requested one k step ahead. For products
// with many 128x128 tiles that are none of the persistent kernel's (N not a
// multiple of 256, short K): there the other block's MFMAs run through one
// block's prologue, epilogue and barriers, which the ring kernel, alone on its
// CU, does not have: 66500 rows of N 1152, K 384 143 us on the ring, 130 here;
// N 384, K 128 38.7, 32.9. Also
// for weights of 2^31 elements and more (64-bit addresses). Sums in the order of
// the other kernels.
constexpr int GM = 128, GN = 128, GK = kRingK, GLD = GK + 8;

template <int EPI>
__global__ __launch_bounds__(256, 2) void gemm_bf16_pair(const bf16* __restrict__ A, int lda,
                                                         const bf16* __restrict__ Bt, const float* __restrict__ bias,
                                                         const void* __restrict__ R, int ldr, void* __restrict__ C,
                                                         int ldc, int M, int N, int K, int tiles_m1, int tiles_m,
                                                         int tiles_n, LnResid ln) {
  __shared__ __attribute__((aligned(16))) bf16 sA[2][GM * GLD];
  __shared__ __attribute__((aligned(16))) bf16 sB[2][GN * GLD];

  const int n_tiles = tiles_m * tiles_n, per_xcd = (n_tiles + 7) >> 3;
  const int t = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (t >= n_tiles) return;
  const int mt = t / tiles_n, n0 = (t % tiles_n) * GN;
  // row tiles from tiles_m1 on lie in the second array (see LnResid::a2)
  const bool second = mt >= tiles_m1;
  const int row0 = second ? ln.m1 : 0;                        // output row of the array's row 0
  const int rows = second ? M - ln.m1 : (ln.a2 ? ln.m1 : M);  // rows of the array
  const int m0 = (second ? mt - tiles_m1 : mt) * GM;
  const bf16* const Ar = second ? (const bf16*)ln.a2 : A;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int l32 = lane & 31, hi = lane >> 5;

  // 128 rows x 8 chunks of 16 B per operand, 4 chunks per thread (rows past the
  // array's last repeat it; their results are not stored)
  bf16x8 ra[4], rb[4];
  auto gload = [&](int k0) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = tid + 256 * u, r = c >> 3, col = (c & 7) * 8;
      ra[u] = *reinterpret_cast<const bf16x8*>(Ar + (size_t)min(m0 + r, rows - 1) * lda + k0 + col);
      rb[u] = *reinterpret_cast<const bf16x8*>(Bt + (size_t)(n0 + r) * K + k0 + col);
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int c = tid + 256 * u, r = c >> 3, col = (c & 7) * 8;
      *reinterpret_cast<bf16x8*>(&sA[buf][r * GLD + col]) = ra[u];
      *reinterpret_cast<bf16x8*>(&sB[buf][r * GLD + col]) = rb[u];
    }
  };

  floatx16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  const int nk = K / GK;
  gload(0);
  lstore(0);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) gload((kt + 1) * GK);
#pragma unroll
    for (int ks = 0; ks < GK / 16; ++ks) {
      bf16x8 fw[2], fx[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fw[i] = *reinterpret_cast<const bf16x8*>(&sB[cur][(wn * 64 + i * 32 + l32) * GLD + ks * 16 + hi * 8]);
        fx[i] = *reinterpret_cast<const bf16x8*>(&sA[cur][(wm * 64 + i * 32 + l32) * GLD + ks * 16 + hi * 8]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (epi_lnfold(EPI))  // fp16 operands (see gemm_bf16_p4)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, fw[i]),
                                                               __builtin_bit_cast(f16x8, fx[j]), acc[i][j], 0, 0, 0);
          else
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[i], fx[j], acc[i][j], 0, 0, 0);
        }
    }
    if (kt + 1 < nk) lstore(cur ^ 1);
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int m = m0 + wm * 64 + j * 32 + l32;
    if (m >= rows) continue;
    const bf16* rrow = (const bf16*)(second ? ln.r2 : R) + (size_t)m * ldr;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      store_acc<EPI>(acc[i][j], row0 + m, n0 + wn * 64 + i * 32 + 4 * hi, bias, rrow, C, ldc, ln);
  }
}

constexpr int kGroupM = 8;  // row blocks that share each column block in turn (L2 reuse)

// Persistent four-wave kernel: one block per CU walks a run of 256x256 output
// tiles. Four waves (one per SIMD) as 2x2, each wave 128x128 of C from 4x4
// v_mfma_f32_32x32x16_bf16 tiles with the fp32 accumulators in AGPRs, so every
// 1 KB fragment read from LDS feeds four MFMAs. K advances 64 at a time through
// two LDS stages (A and B tiles of 128-byte rows; 16-byte slot s of row r is
// held at slot s ^ ((r / 2) % 8), so row-wise stores and column-wise fragment
// reads are both free of bank conflicts without padding).
//
// Operands travel global -> registers -> LDS in four groups of 64 bytes per
// thread. Group q >= 1 of k step t + 1 is parked during sub-step q - 1 of step t
// and group 0 of step t + 2 during its sub-step 3 (right after the barrier that
// frees the stage), each group being refetched as soon as it is parked: every
// load has one whole k step of MFMA work to land, and the loads are spread
// evenly over the step instead of arriving in one burst. The load stream runs
// across tile boundaries and the epilogue parks results in an LDS area of its
// own, so the pipeline never drains between tiles.
constexpr int kPStage = 2 * PT * PK;

#define TX_LGKM_BARRIER() asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory")

template <int EPI>
__global__ __launch_bounds__(256, 1) void gemm_bf16_p4(const bf16* __restrict__ A, int lda,
                                                       const bf16* __restrict__ Bt,
                                                       const float* __restrict__ bias,
                                                       const void* __restrict__ R, int ldr, void* __restrict__ C,
                                                       int ldc, int M, int N, int K, int tiles_m, int tiles_n,
                                                       int n_tiles, int per_xcd, LnResid ln) {
  __shared__ __attribute__((aligned(16))) bf16 lds[2 * kPStage];
  __shared__ __attribute__((aligned(16))) float park_all[4 * 32 * 64];

  const int nloc = gridDim.x >> 3, local = blockIdx.x >> 3;
  const int t_begin = (blockIdx.x & 7) * per_xcd, t_end = min(n_tiles, t_begin + per_xcd);
  const int my_tiles = t_begin + local < t_end ? (t_end - t_begin - local + nloc - 1) / nloc : 0;
  if (my_tiles == 0) return;
  const int nk = K / PK;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int l32 = lane & 31, hi = lane >> 5;

  auto tile_origin = [&](int i, int& m0, int& n0) {
    const int t = t_begin + local + min(i, my_tiles - 1) * nloc;
    const int group = t / (kGroupM * tiles_n);
    const int first_m = group * kGroupM;
    const int gm_size = min(tiles_m - first_m, kGroupM);
    m0 = (first_m + (t % (kGroupM * tiles_n)) % gm_size) * PT;
    n0 = ((t % (kGroupM * tiles_n)) / gm_size) * PT;
  };

  // staging: chunk u of this thread is row (tid / 8) + 32 u, 16-byte slot
  // tid % 8 of both operand tiles; group q holds chunks 2q and 2q + 1
  const int srow = tid >> 3, sslot = tid & 7;
  const int wofs = srow * PK + ((sslot ^ ((srow >> 1) & 7)) << 3);
  bf16x8 ga[8], gb[8];
  // Operands through raw buffer loads: the lane's byte offset within a tile is
  // fixed (row srow + 32 u, slot sslot), the tile's row base is added as one
  // 32-bit value and k0 travels in the scalar offset. Rows past M fall beyond
  // the A resource's extent and read as zeros; their results are not stored.
  // (extents in bytes: the launcher keeps M lda and N K below 2^31 elements;
  // word 3 of the resource as CDNA wants it for raw loads)
  const __amdgpu_buffer_rsrc_t ra =
      __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, (int)(2u * (uint32_t)M * (uint32_t)lda), 0x00020000);
  const __amdgpu_buffer_rsrc_t rb =
      __builtin_amdgcn_make_buffer_rsrc((void*)Bt, 0, (int)(2u * (uint32_t)N * (uint32_t)K), 0x00020000);
  const uint32_t la = 2u * (uint32_t)(srow * lda + sslot * 8), lb = 2u * (uint32_t)(srow * K + sslot * 8);
  auto gload = [&](auto Q_, int m0, int n0, int k0) {
    constexpr int Q = decltype(Q_)::value;
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int u = 2 * Q + v;
      const uint32_t oa = 2u * ((uint32_t)(m0 + 32 * u) * (uint32_t)lda) + la;
      const uint32_t ob = 2u * ((uint32_t)(n0 + 32 * u) * (uint32_t)K) + lb;
      ga[u] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)oa, 2 * k0, 0));
      gb[u] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rb, (int)ob, 2 * k0, 0));
    }
  };
  auto lstore = [&](auto Q_, int stage) {
    constexpr int Q = decltype(Q_)::value;
    bf16* sa = lds + stage * kPStage;
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int u = 2 * Q + v;
      *reinterpret_cast<bf16x8*>(sa + wofs + u * 32 * PK) = ga[u];
      *reinterpret_cast<bf16x8*>(sa + PT * PK + wofs + u * 32 * PK) = gb[u];
    }
  };

  // fragment reads: A rows wm*128 + 32 j + l32, B rows wn*128 + 32 i + l32;
  // k sub-step ks covers slots 2 ks + hi
  int rofs[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) rofs[ks] = l32 * PK + (((2 * ks + hi) ^ ((l32 >> 1) & 7)) << 3);
  const int a_base = wm * 128 * PK, b_base = PT * PK + wn * 128 * PK;
  auto fread = [&](bf16x8(&fa)[4], bf16x8(&fb)[4], int stage, int ks) {
    const bf16* s = lds + stage * kPStage;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      fa[q] = *reinterpret_cast<const bf16x8*>(s + a_base + q * 32 * PK + rofs[ks]);
      fb[q] = *reinterpret_cast<const bf16x8*>(s + b_base + q * 32 * PK + rofs[ks]);
    }
  };

  floatx16 acc[4][4];
  bf16x8 fa0[4], fb0[4], fa1[4], fb1[4];
  // the LayerNorm-folding epilogues take fp16 operands (the stored pre-LN sum
  // and the gain-scaled weight); the fragments are the same 16-byte units
  auto mfma16 = [&](auto Z_, const bf16x8(&fa)[4], const bf16x8(&fb)[4]) {
    constexpr bool Z = decltype(Z_)::value;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (epi_lnfold(EPI))
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, fb[i]),
                                                             __builtin_bit_cast(f16x8, fa[j]),
                                                             Z ? floatx16{} : acc[i][j], 0, 0, 0);
        else
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[i], fa[j], Z ? floatx16{} : acc[i][j], 0, 0, 0);
      }
  };
  using F0 = std::false_type;
  using T1 = std::true_type;
  // 16 MFMAs with 8 fragment reads, 4 LDS stores and 4 global loads between
  // them: the reads (the next sub-step's fragments) between the first eight
  // MFMAs, so that they have the second half to land, then the stores and
  // loads (~1% faster than spreading the reads over all sixteen)
  auto interleave = [&]() {
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  using I0 = std::integral_constant<int, 0>;
  using I1 = std::integral_constant<int, 1>;
  using I2 = std::integral_constant<int, 2>;
  using I3 = std::integral_constant<int, 3>;

  // tile-local k step -> (tile origin, column): steps past the tile belong to
  // the next one (the last tile stands in for a next tile that does not exist)
  int m0, n0, nm0, nn0;
  auto target = [&](int kt, int& tm0, int& tn0, int& k0) {
    const bool nxt = kt >= nk;
    tm0 = nxt ? nm0 : m0;
    tn0 = nxt ? nn0 : n0;
    k0 = (nxt ? kt - nk : kt) * PK;
  };

  // One k step on stage S (= kt % 2); see the kernel comment for the order
  auto step = [&](auto S_, auto Z_, int kt) {
    constexpr int S = decltype(S_)::value;
    int am0, an0, ak0, bm0, bn0, bk0;
    target(kt + 2, am0, an0, ak0);
    target(kt + 3, bm0, bn0, bk0);
    fread(fa1, fb1, S, 1);
    lstore(I1{}, S ^ 1);
    gload(I1{}, am0, an0, ak0);
    mfma16(Z_, fa0, fb0);
    interleave();
    fread(fa0, fb0, S, 2);
    lstore(I2{}, S ^ 1);
    gload(I2{}, am0, an0, ak0);
    mfma16(F0{}, fa1, fb1);
    interleave();
    fread(fa1, fb1, S, 3);
    lstore(I3{}, S ^ 1);
    gload(I3{}, am0, an0, ak0);
    mfma16(F0{}, fa0, fb0);
    interleave();
    TX_LGKM_BARRIER();
    fread(fa0, fb0, S ^ 1, 0);
    lstore(I0{}, S);
    gload(I0{}, bm0, bn0, bk0);
    mfma16(F0{}, fa1, fb1);
    interleave();
  };

  // prologue: stage 0 = step 0, group 0 of step 1 in stage 1; registers hold
  // group 0 of step 2 and groups 1..3 of step 1
  tile_origin(0, m0, n0);
  tile_origin(1, nm0, nn0);
  {
    int tm0, tn0, k0;
    gload(I0{}, m0, n0, 0);
    gload(I1{}, m0, n0, 0);
    gload(I2{}, m0, n0, 0);
    gload(I3{}, m0, n0, 0);
    lstore(I0{}, 0);
    lstore(I1{}, 0);
    lstore(I2{}, 0);
    lstore(I3{}, 0);
    target(1, tm0, tn0, k0);
    gload(I0{}, tm0, tn0, k0);
    lstore(I0{}, 1);
    gload(I1{}, tm0, tn0, k0);
    gload(I2{}, tm0, tn0, k0);
    gload(I3{}, tm0, tn0, k0);
    target(2, tm0, tn0, k0);
    gload(I0{}, tm0, tn0, k0);
  }
  TX_LGKM_BARRIER();
  fread(fa0, fb0, 0, 0);

  float* park = park_all + wave * 32 * 64;
  const int er = lane >> 3, ec = lane & 7;  // row (plus 8 u) and 8-float chunk of the read-back
  // epilogue resources (extents in bytes, below 2^32: checked by the launcher)
  // and the lane's fixed offsets: row wm * 128 + er (+ 32 j + 8 u), column
  // wn * 128 + 8 ec (+ 64 h) of the tile, and the LayerNorm statistics of the
  // same rows
  constexpr bool kStats = EPI == EPI_BIAS_RESLN || epi_lnfold(EPI);  // row statistics used
  const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)R, 0, epi_resid(EPI) ? (int)(2u * (uint32_t)M * (uint32_t)ldr) : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)ln.stats, 0, kStats ? (int)(8u * (uint32_t)M) : 0, 0x00020000);
  const __amdgpu_buffer_rsrc_t rc =
      __builtin_amdgcn_make_buffer_rsrc(C, 0, (int)(2u * (uint32_t)M * (uint32_t)ldc), 0x00020000);
  const uint32_t lr = 2u * (uint32_t)((wm * 128 + er) * ldr + wn * 128 + ec * 8);
  const uint32_t lc = 2u * (uint32_t)((wm * 128 + er) * ldc + wn * 128 + ec * 8);
  const uint32_t ls = 8u * (uint32_t)(wm * 128 + er);

  for (int i = 0; i < my_tiles; ++i) {
    // the tile's first MFMAs take a zero accumulator input
    step(I0{}, T1{}, 0);
    step(I1{}, F0{}, 1);
    for (int kt = 2; kt < nk; kt += 2) {
      step(I0{}, F0{}, kt);
      step(I1{}, F0{}, kt + 1);
    }
    const int cm0 = m0, cn0 = n0;
    m0 = nm0;
    n0 = nn0;
    tile_origin(i + 2, nm0, nn0);

    // epilogue: per round each wave parks 32 rows x 64 columns of fp32 results
    // (16-byte unit q of row r at unit q ^ (r % 16): conflict-free both ways)
    // and reads them back row-contiguously, 8 lanes per 128-byte row segment;
    // bias, GELU or residual applied with one rounding (bf16, or fp16 for a
    // pre-LN sum). Rows past M (computed from zero rows) are not stored.
    // Rounds (j, h): 32 rows (32 j ..) x 64 columns (64 h ..) of the wave's
    // 128 x 128. The residual pieces of a round are fetched one round ahead,
    // and the LayerNorm statistics of the lane's four rows (shared by both
    // rounds of j) a j ahead, each lane loading its own rows' (a broadcast
    // within the load: no lane permutes). The column vectors (bias, and for a
    // LayerNorm residual its gain and offset, the offset folded into the bias;
    // for a folded LayerNorm the weight's column sums) are read again each
    // round (L1 hits) rather than held through the epilogue. Residual, statistics
    // and outputs go through raw buffer operations with 32-bit offsets: rows
    // past M lie beyond the resources, read as zeros and are not written.
    u32x4 rres[4];
    LnRow stn[4], stc[4];  // statistics of the lane's rows er + 8 u (next j, current j)
    auto rload = [&](int j, int h) {
      if (epi_resid(EPI)) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t o = 2u * ((uint32_t)(cm0 + j * 32 + 8 * u) * (uint32_t)ldr + (uint32_t)(cn0 + 64 * h)) + lr;
          rres[u] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rr, (int)o, 0, 0));
        }
      }
      if (kStats && h == 0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const uint32_t o = 8u * (uint32_t)(cm0 + j * 32 + 8 * u) + ls;
          const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)o, 0, 0));
          stn[u] = LnRow{__uint_as_float(v[0]), __uint_as_float(v[1])};
        }
      }
    };
    rload(0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const floatx4 v4 = {acc[2 * h + ii][j][4 * g], acc[2 * h + ii][j][4 * g + 1], acc[2 * h + ii][j][4 * g + 2],
                                acc[2 * h + ii][j][4 * g + 3]};
            const int q = ii * 8 + 2 * g + hi;
            *reinterpret_cast<floatx4*>(park + l32 * 64 + ((q ^ (l32 & 15)) << 2)) = v4;
          }
        u32x4 rcur[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) rcur[u] = rres[u];
        if (h == 0)
#pragma unroll
          for (int u = 0; u < 4; ++u) stc[u] = stn[u];
        if (j * 2 + h + 1 < 8) rload((j * 2 + h + 1) >> 1, (j * 2 + h + 1) & 1);
        asm volatile("" ::: "memory");  // keeps the column vectors from being held across rounds
        const int ncol = cn0 + wn * 128 + 64 * h + ec * 8;
        floatx4 cb[2], lg[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          cb[q] = *reinterpret_cast<const floatx4*>(bias + ncol + 4 * q);
          if (EPI == EPI_BIAS_RESLN) cb[q] += *reinterpret_cast<const floatx4*>(ln.b + ncol + 4 * q);
          if (kStats) lg[q] = *reinterpret_cast<const floatx4*>(ln.g + ncol + 4 * q);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int r = er + 8 * u;
          const floatx4 x0 = *reinterpret_cast<const floatx4*>(park + r * 64 + (((2 * ec) ^ (r & 15)) << 2));
          const floatx4 x1 = *reinterpret_cast<const floatx4*>(park + r * 64 + (((2 * ec + 1) ^ (r & 15)) << 2));
          const uint32_t o_off = 2u * ((uint32_t)(cm0 + j * 32 + 8 * u) * (uint32_t)ldc + (uint32_t)(cn0 + 64 * h)) + lc;
          u32x4 ov;
          if (epi_lnfold(EPI)) {
            // LN(A) W + b = (acc * x + y * cs) + b' for the row's statistics (x, y)
            const LnRow st = stc[u];
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              float v0 = fmaf(x0[e], st.x, fmaf(st.y, lg[0][e], cb[0][e]));
              float v1 = fmaf(x1[e], st.x, fmaf(st.y, lg[1][e], cb[1][e]));
              if (epi_gelu(EPI)) {
                v0 = gelu_erf(v0);
                v1 = gelu_erf(v1);
              }
              o[e] = (bf16)v0;
              o[e + 4] = (bf16)v1;
            }
            ov = __builtin_bit_cast(u32x4, o);
          } else if (epi_resid(EPI)) {
            LnRow st{0.f, 0.f};
            if (EPI == EPI_BIAS_RESLN) st = stc[u];
            f16x8 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float r0 = resid8<EPI>(rcur[u], e, st, EPI == EPI_BIAS_RESLN ? lg[0][e] : 0.f);
              const float r1 = resid8<EPI>(rcur[u], e + 4, st, EPI == EPI_BIAS_RESLN ? lg[1][e] : 0.f);
              o[e] = (f16)epilogue<EPI>(x0[e], cb[0][e], r0);
              o[e + 4] = (f16)epilogue<EPI>(x1[e], cb[1][e], r1);
            }
            ov = __builtin_bit_cast(u32x4, o);
          } else {
            bf16x8 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              o[e] = (bf16)epilogue<EPI>(x0[e], cb[0][e], 0.f);
              o[e + 4] = (bf16)epilogue<EPI>(x1[e], cb[1][e], 0.f);
            }
            ov = __builtin_bit_cast(u32x4, o);
          }
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, ov),
                                                 rc, (int)o_off, 0, 0);
        }
      }
  }
}

// Plain tiled GEMM for shapes and alignments the MFMA kernels do not cover:
// 64x64 block tile, K step 16, each thread computes 4x4 outputs in fp32.
// Sum type (pre-LN sums of the residual epilogues): fp16 beside bf16, fp32
// beside fp32.
template <typename T>
using SumT = typename std::conditional<std::is_same<T, float>::value, float, f16>::type;

template <typename T, int EPI>
__global__ __launch_bounds__(256) void gemm_plain(const T* __restrict__ A, int lda, const T* __restrict__ Bt,
                                                  const float* __restrict__ bias, const void* __restrict__ R, int ldr,
                                                  void* __restrict__ C, int ldc, int M, int N, int K, LnResid ln) {
  typedef SumT<T> S;
  typedef typename std::conditional<EPI == EPI_BIAS_RESLN, S, T>::type RT;  // residual element type
  typedef typename std::conditional<epi_resid(EPI), S, T>::type CT;  // output element type
  __shared__ float sA[16][64 + 4];
  __shared__ float sB[16][64 + 4];
  const int m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = tid + 256 * u, r = e >> 4, c = e & 15;
      const int gm = m0 + r, gn = n0 + r, gk = k0 + c;
      sA[c][r] = (gm < M && gk < K) ? (float)A[(size_t)gm * lda + gk] : 0.f;
      sB[c][r] = (gn < N && gk < K) ? (float)Bt[(size_t)gn * K + gk] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = sA[kk][ty * 4 + i];
        b[i] = sB[kk][tx * 4 + i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }
  const RT* Rt = (const RT*)R;
  CT* Ct = (CT*)C;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
    LnRow st{0.f, 0.f};
    if (EPI == EPI_BIAS_RESLN) st = ln.stats[m];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= N) continue;
      float r = 0.f, bn = bias[n];
      if (EPI == EPI_BIAS_RESID) r = (float)Rt[(size_t)m * ldr + n];
      if (EPI == EPI_BIAS_RESLN) {
        r = ln_resid((float)Rt[(size_t)m * ldr + n], st, ln.g[n]);
        bn += ln.b[n];
      }
      Ct[(size_t)m * ldc + n] = (CT)epilogue<EPI>(acc[i][j], bn, r);
    }
  }
}

// fp32 models: v_mfma_f32_16x16x4_f32, one wave per TM x TN tiles of 16x16
// outputs, four waves per block on adjacent column tiles, no LDS. A lane loads
// 16 bytes of its A and B rows per 16 columns of k; the MFMA of element t sums
// k = 4 (lane / 16) + t, the same columns on both operands. What bounds the
// fp32 model's few rows is latency (loads, then 4 MFMAs per 16 columns), which
// small tiles over many CUs and four chunks in flight keep short: M 24, K 64
// or 256 9-18 us per launch on gemm_plain (64x64 tiles through LDS, a barrier
// per 16 columns), 3-6 here. 32x32 outputs per wave once those fill the CUs
// (half the operand reads); both sum each output in the same order.
template <int EPI, int TM, int TN>
__global__ __launch_bounds__(256) void gemm_f32_mfma(const float* __restrict__ A, int lda, const float* __restrict__ Bt,
                                                     const float* __restrict__ bias, const float* __restrict__ R,
                                                     int ldr, float* __restrict__ C, int ldc, int M, int N, int K,
                                                     LnResid ln) {
  const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  const int m0 = blockIdx.y * (16 * TM), n0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * (16 * TN);
  if (n0 >= N) return;  // whole waves; the kernel has no barrier
  const float *ap[TM], *bp[TN];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int m = min(m0 + 16 * i + l16, M - 1);
    ap[i] = (ln.a2 && m >= ln.m1 ? (const float*)ln.a2 + (size_t)(m - ln.m1) * lda : A + (size_t)m * lda) + 4 * g;
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) bp[j] = Bt + (size_t)min(n0 + 16 * j + l16, N - 1) * K + 4 * g;
  // even and odd chunks sum apart: two chains of half the length
  floatx4 acc[TM][TN], odd[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = odd[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  constexpr int D = 4;  // chunks of 16 columns in flight
  floatx4 a[D][TM], b[D][TN];
  auto load = [&](int s, int k0) {
#pragma unroll
    for (int i = 0; i < TM; ++i) a[s][i] = *reinterpret_cast<const floatx4*>(ap[i] + k0);
#pragma unroll
    for (int j = 0; j < TN; ++j) b[s][j] = *reinterpret_cast<const floatx4*>(bp[j] + k0);
  };
#pragma unroll
  for (int s = 0; s < D; ++s)
    if (16 * s < K) load(s, 16 * s);
  for (int k0 = 0; k0 < K; k0 += 16 * D)
#pragma unroll
    for (int s = 0; s < D; ++s) {
      if (k0 + 16 * s >= K) break;
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            floatx4& c = s & 1 ? odd[i][j] : acc[i][j];
            c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s][i][t], b[s][j][t], c, 0, 0, 0);
          }
      if (k0 + 16 * (s + D) < K) load(s, k0 + 16 * (s + D));
    }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] += odd[i][j];
  // accumulator element v of tile (i, j): row m0 + 16 i + 4 g + v, column n0 + 16 j + l16
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n0 + 16 * j + l16;
    if (n >= N) continue;
    float bn = bias[n], gn = 0.f;
    if (EPI == EPI_BIAS_RESLN) {
      bn += ln.b[n];
      gn = ln.g[n];
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = m0 + 16 * i + 4 * g + v;
        if (m >= M) continue;
        float r = 0.f;
        if (epi_resid(EPI))
          r = ln.a2 && m >= ln.m1 ? ((const float*)ln.r2)[(size_t)(m - ln.m1) * ldr + n] : R[(size_t)m * ldr + n];
        if (EPI == EPI_BIAS_RESLN) r = ln_resid(r, ln.stats[m], gn);
        C[(size_t)m * ldc + n] = epilogue<EPI>(acc[i][j][v], bn, r);
      }
  }
}

template <int TM, int TN>
static hipError_t f32_mfma(const float* A, int lda, const float* Bt, const float* bias, const float* R, int ldr, float* C,
                           int ldc, int M, int N, int K, Epilogue epi, LnResid ln, hipStream_t s) {
  const dim3 grid((N + 64 * TN - 1) / (64 * TN), (M + 16 * TM - 1) / (16 * TM));
#define TX_F32(E) gemm_f32_mfma<E, TM, TN><<<grid, 256, 0, s>>>(A, lda, Bt, bias, R, ldr, C, ldc, M, N, K, ln)
  switch (epi) {
    case EPI_BIAS: TX_F32(EPI_BIAS); break;
    case EPI_BIAS_GELU: TX_F32(EPI_BIAS_GELU); break;
    case EPI_BIAS_RESID: TX_F32(EPI_BIAS_RESID); break;
    case EPI_BIAS_RESLN: TX_F32(EPI_BIAS_RESLN); break;
    default: return hipErrorInvalidValue;  // the LayerNorm-folding epilogues are for bf16 models
  }
#undef TX_F32
  return hipGetLastError();
}

template <typename T>
static hipError_t plain(const void* A, int lda, const void* Bt, const float* bias, const void* R, int ldr, void* C,
                        int ldc, int M, int N, int K, Epilogue epi, LnResid ln, hipStream_t s) {
  dim3 grid((N + 63) / 64, (M + 63) / 64);
  const T* a = (const T*)A;
  const T* b = (const T*)Bt;
#define TX_PL(E) gemm_plain<T, E><<<grid, 256, 0, s>>>(a, lda, b, bias, R, ldr, C, ldc, M, N, K, ln)
  switch (epi) {
    case EPI_BIAS: TX_PL(EPI_BIAS); break;
    case EPI_BIAS_GELU: TX_PL(EPI_BIAS_GELU); break;
    case EPI_BIAS_RESID: TX_PL(EPI_BIAS_RESID); break;
    case EPI_BIAS_RESLN: TX_PL(EPI_BIAS_RESLN); break;
    default: return hipErrorInvalidValue;  // the LayerNorm-folding epilogues run on the MFMA kernels only
  }
#undef TX_PL
  return hipGetLastError();
}

bool gemm_ln_ok(int N, int K, int lda, int ldc) {
  return N % 128 == 0 && K % kRingK == 0 && lda % 8 == 0 && ldc % 8 == 0;
}

hipError_t launch_gemm(bool bf, const void* A, int lda, const void* Bt, const float* bias, const void* R, int ldr,
                       void* C, int ldc, int M, int N, int K, Epilogue epi, hipStream_t s, LnResid ln) {
  if (M <= 0) return hipSuccess;
  if (epi == EPI_BIAS_RESLN && (!ln.stats || !ln.g || !ln.b)) return hipErrorInvalidValue;
  if (epi_resid(epi) && !R) return hipErrorInvalidValue;
  if (epi_lnfold(epi) && (!bf || !ln.stats || !ln.g || !gemm_ln_ok(N, K, lda, ldc))) return hipErrorInvalidValue;
  // rows of two arrays on a kernel that takes one: a launch for each
  auto halves = [&]() {
    LnResid l1 = ln, l2 = ln;
    l1.a2 = l1.r2 = l2.a2 = l2.r2 = nullptr;
    l1.m1 = l2.m1 = 0;
    if (l2.stats) l2.stats += ln.m1;
    const size_t es = bf ? 2 : 4;
    const hipError_t e = launch_gemm(bf, A, lda, Bt, bias, R, ldr, C, ldc, ln.m1, N, K, epi, s, l1);
    if (e != hipSuccess) return e;
    return launch_gemm(bf, ln.a2, lda, Bt, bias, ln.r2, ldr, (char*)C + (size_t)ln.m1 * ldc * es, ldc, M - ln.m1, N, K,
                       epi, s, l2);
  };
  if (ln.a2 && (ln.m1 < 0 || ln.m1 > M || (epi_resid(epi) && !ln.r2))) return hipErrorInvalidValue;
  auto row_range = [&](long long m0, int mc) {  // rows m0 .. m0 + mc - 1 of one array
    LnResid lc = ln;
    if (lc.stats) lc.stats += m0;
    const size_t es = bf ? 2 : 4;
    return launch_gemm(bf, (const char*)A + m0 * lda * es, lda, Bt, bias,
                       R ? (const void*)((const char*)R + m0 * ldr * es) : nullptr, ldr, (char*)C + m0 * ldc * es, ldc,
                       mc, N, K, epi, s, lc);
  };
  auto row_ranges = [&](long long rows_max) {
    for (long long m0 = 0; m0 < M; m0 += rows_max) {
      const hipError_t e = row_range(m0, (int)std::min(rows_max, (long long)M - m0));
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  };
  if (!bf) {
    // 16-byte operand loads: K a multiple of a chunk, rows and bases aligned (a
    // caller's tokens may be aligned to 4 bytes only)
    if (K % 16 == 0 && lda % 4 == 0 && (((uintptr_t)A | (uintptr_t)Bt | (uintptr_t)ln.a2) & 15) == 0) {
      constexpr int kGridRows = 16 * 65535;  // the grid's y extent
      if (M > kGridRows) return ln.a2 ? halves() : row_ranges(kGridRows);
      const float *a = (const float*)A, *b = (const float*)Bt, *r = (const float*)R;
      if ((long long)((M + 31) / 32) * ((N + 31) / 32) >= 1024)  // four waves on each of 256 CUs
        return f32_mfma<2, 2>(a, lda, b, bias, r, ldr, (float*)C, ldc, M, N, K, epi, ln, s);
      return f32_mfma<1, 1>(a, lda, b, bias, r, ldr, (float*)C, ldc, M, N, K, epi, ln, s);
    }
    if (ln.a2) return halves();
    return plain<float>(A, lda, Bt, bias, R, ldr, C, ldc, M, N, K, epi, ln, s);
  }
  // The MFMA kernels address A, R and C with 32-bit byte offsets: a product
  // whose operands span 2^31 elements or more runs as several row chunks.
  {
    const long long ld_max = std::max({(long long)lda, (long long)ldc, epi_resid(epi) ? (long long)ldr : 1ll});
    const long long rows_max = std::max(256ll, ((1ll << 31) - 1) / ld_max / 256 * 256);
    if (M > rows_max) return ln.a2 ? halves() : row_ranges(rows_max);
  }
  const bool aligned = (lda % 8 == 0) && (ldc % 8 == 0) && (ldr % 8 == 0) && (((uintptr_t)A & 15) == 0) &&
                       (((uintptr_t)Bt & 15) == 0) && (((uintptr_t)C & 15) == 0) && (((uintptr_t)R & 15) == 0) &&
                       (((uintptr_t)bias & 15) == 0) && (((uintptr_t)ln.g & 15) == 0) &&
                       (((uintptr_t)ln.b & 15) == 0) && ((((uintptr_t)ln.a2 | (uintptr_t)ln.r2) & 15) == 0);
  const bool mfma = N % 128 == 0 && K % kRingK == 0 && aligned;
  if (ln.a2 && !mfma) return halves();
  if (!mfma)
    return plain<bf16>(A, lda, Bt, bias, R, ldr, C, ldc, M, N, K, epi, ln, s);
  const bf16* a = (const bf16*)A;
  const bf16* b = (const bf16*)Bt;
  // the current device's CU count, looked up once per device
  static std::atomic<int> cu_of_device[64];
  int dev = 0, n_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = -1;
  if (dev >= 0) n_cu = cu_of_device[dev].load(std::memory_order_relaxed);
  if (n_cu <= 0) {
    if (dev < 0 || hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 8)
      n_cu = 256;
    if (dev >= 0) cu_of_device[dev].store(n_cu, std::memory_order_relaxed);
  }
  const bool persistent = persistent_shape(M, N, K, std::max({(long long)lda, (long long)ldc, (long long)ldr}));
  const int tile = pick_tile(M, N, K, persistent, n_cu);
  if (ln.a2 && tile == kPersistent) return halves();
  if (tile == kPersistent) {
    const int m1 = persistent_rows(M, N, K, n_cu);
    if (m1 < M) {
      const hipError_t e = row_range(0, m1);
      return e != hipSuccess ? e : row_range(m1, M - m1);
    }
  }
  const int bm = kTileCost[tile].bm, tiles_n = N / kTileCost[tile].bn;
  const int tiles_m1 = ((ln.a2 ? ln.m1 : M) + bm - 1) / bm, tiles_m = tiles_m1 + (ln.a2 ? (M - ln.m1 + bm - 1) / bm : 0);
  const int n_tiles = tiles_n * tiles_m, per_xcd = (n_tiles + 7) / 8;
#define TX_GP4(E)                                                                                               \
  gemm_bf16_p4<E><<<8 * std::max(1, std::min(n_cu / 8, per_xcd)), 256, 0, s>>>(a, lda, b, bias, R, ldr, C, ldc, M, N, \
                                                                              K, tiles_m, tiles_n, n_tiles, per_xcd, ln)
  // tiles in column order when the weight is the larger operand (each XCD then
  // reads a part of it), in row order otherwise
#define TX_GR(E, BM, BN, MI, NI, S)                                                                                  \
  gemm_bf16_ring<E, BM, BN, MI, NI, S><<<8 * per_xcd, 256, 0, s>>>(a, lda, b, bias, R, ldr, C, ldc, M, N, K, tiles_m1, \
                                                                   tiles_m, tiles_n, M <= N, ln)
#define TX_GPAIR(E)                                                                                                   \
  gemm_bf16_pair<E><<<8 * per_xcd, 256, 0, s>>>(a, lda, b, bias, R, ldr, C, ldc, M, N, K, tiles_m1, tiles_m, tiles_n, \
                                                ln)
#define TX_GT(E)                                          \
  switch (tile) {                                         \
    case T32x32: TX_GR(E, 32, 32, 1, 1, 16); break;       \
    case T32x64: TX_GR(E, 32, 64, 1, 1, 6); break;        \
    case T64x64: TX_GR(E, 64, 64, 1, 1, 4); break;        \
    case T64x128: TX_GR(E, 64, 128, 1, 2, 6); break;      \
    case T128x128: TX_GR(E, 128, 128, 2, 2, 4); break;    \
    case kPair: TX_GPAIR(E); break;                       \
    default: TX_GP4(E); break;                            \
  }
  switch (epi) {
    case EPI_BIAS: TX_GT(EPI_BIAS); break;
    case EPI_BIAS_GELU: TX_GT(EPI_BIAS_GELU); break;
    case EPI_BIAS_RESID: TX_GT(EPI_BIAS_RESID); break;
    case EPI_BIAS_RESLN: TX_GT(EPI_BIAS_RESLN); break;
    case EPI_LN: TX_GT(EPI_LN); break;
    case EPI_LN_GELU: TX_GT(EPI_LN_GELU); break;
  }
#undef TX_GT
#undef TX_GPAIR
#undef TX_GR
#undef TX_GP4
  return hipGetLastError();
}

}  // namespace tx
