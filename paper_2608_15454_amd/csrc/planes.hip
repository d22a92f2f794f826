// gfx950 matrix products on split rows.
//
// Long passes (prefill, the full-sequence forward) keep the input of every linear layer
// as bfloat16 halves, hi = bf16(x) and lo = bf16(x - hi), interleaved in groups of 32
// columns: the split that the matrix cores need anyway, made once by the kernel that
// produces the rows instead of once per column tile by every block that reads them.  The product kernel then moves bytes only.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <math.h>

#include <algorithm>
#include <type_traits>

#include "dev.h"
#include "kernels.h"

namespace mbp {
namespace {

using namespace dev;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

template <typename Kern, typename... Args>
hipError_t plaunch(Kern kernel, dim3 grid, dim3 block, hipStream_t st, hipEvent_t e0, hipEvent_t e1, Args... args) {
  if (e0 != nullptr || e1 != nullptr) {
    hipExtLaunchKernelGGL(kernel, grid, block, 0, st, e0, e1, 0, args...);
  } else {
    hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
  }
  return hipGetLastError();
}

constexpr int kBK = 32;
constexpr int kPlanesMinRows = 65;

// One output tile of BM x BN per block of WM x WN waves, each wave TI x TJ blocks of
// v_mfma_f32_32x32x16_bf16, K in steps of 32.  LDS holds three steps of X (BM rows of 64
// bytes hi, 64 bytes lo) and two double steps of the weights (BN rows of 128 bytes): all
// 160 KB of a compute unit for one 256 x 256 tile (eight waves of 64 rows x 128 columns)
// or two 128 x 128 tiles (four waves of 64 x 64).
//
// Bound by the matrix cores, at the clock their power leaves: two MFMAs per product keep
// them busy 65 % of the cycles (SQ_VALU_MFMA_BUSY_CYCLES over the 256 tile's launches in
// prompts of 131072 rows) at 1.72 GHz.  Against a
// tile that read float32 rows, split them in every block and staged them through
// registers (44-48 % busy), at M = 131072, d = 1024: gate/up 4093 -> 3366 us (653
// TFLOP/s), down 2072 -> 1658 (663), output 669 -> 591, QKV 2181 -> 1730; at M = 32768,
// d = 2048 down runs at 720.  What it took, gate/up at M = 131072:
// - loads straight to LDS and no conversion: 3850 us;
// - LDS reads and loads spread between the MFMAs, banks free of conflicts: 3630;
// - 128-byte rows for every load, hi and lo halves side by side: 3366 (64-byte pieces of
//   16 rows per load held the L2 requests at twice their number).
template <int WM, int WN, int TI, int TJ>
struct PTile {
  static constexpr int NW = WM * WN, BM = 32 * TI * WM, BN = 32 * TJ * WN;
  static constexpr int GA = BM / 8 / NW, GB = BN / 8 / NW;  // 1 KB pieces per wave of a slot
  static constexpr int kA = BM * 128, kW = BN * 128, kLds = 3 * kA + 2 * kW;
  static_assert(GA == 4 && GB == 4, "the wait counts of the loop");
};
using PTile128 = PTile<2, 2, 2, 2>;
using PTile256 = PTile<4, 2, 2, 4>;

// EK: what the kernel ends with, compiled in (an EpiKind, or kEpiPart: the raw sums of a K
// range), since a short launch fetches every line of its code uncached: with one kernel
// for all kinds the 15 us launches of the LM module took 2 to 3 us longer.  kEpiAny: the
// kind at run time, for the 256 tile, whose launches are long and whose epilogues spill
// when compiled alone.
constexpr int kEpiPart = 4, kEpiAny = -1;

template <int WM, int WN, int TI, int TJ, int EK>
__global__ __launch_bounds__(64 * WM * WN, 2) void gemm_planes_kernel(PlaneLinear P) {
  using T = PTile<WM, WN, TI, TJ>;
  constexpr int BM = T::BM, BN = T::BN, GA = T::GA, GB = T::GB;
  __shared__ __attribute__((aligned(1024))) char lds[T::kLds];
  const int kind = EK == kEpiAny ? P.kind : EK;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // The start is kept short (no division, two lines of arguments): a launch of the LM
  // module over a prompt lasts 15 us, and its instructions and arguments start uncached.
  int bx = blockIdx.x, by = blockIdx.y;
  if (P.ginv != 0) {  // XCD k takes groups of 2^grl row blocks k, k + 8, ..., walked rows fastest
    const int bid = by * P.cb + bx, xcd = bid & 7, l = bid >> 3;
    const int g = (int)__umulhi((uint32_t)l, P.ginv), rem = l - ((g * P.cb) << P.grl);
    bx = rem >> P.grl;
    by = xcd + 8 * ((g << P.grl) + (rem & ((1 << P.grl) - 1)));
  }
  const int m0 = by * BM;
  const int K = P.K, M = P.M;
  // this block's steps: K / ksplit columns from z K / ksplit on; nk is even and >= 4
  const int nk = EK == kEpiPart ? K / kBK / P.ksplit : K / kBK;
  const uint32_t kz = EK == kEpiPart ? blockIdx.z * (uint32_t)nk : 0;
  // Piece p of a slot is rows 8 p .. 8 p + 7, eight lanes per row of 128 bytes (a load
  // that covers whole lines moves about three times the bytes of one that takes 64 from
  // each).  A row's 16-byte chunks are stored XOR-ed with (row / 2) % 8, so that the
  // sixteen rows a quarter-wave reads lie in different banks (64 banks of 4 bytes).
  uint32_t va[GA], vb[GB];
  const char* sb[GB];
  const uint32_t ldxb = (uint32_t)P.ldx * 4;
#pragma unroll
  for (int g = 0; g < GA; ++g) {
    const int r = (wave * GA + g) * 8 + (lane >> 3);
    va[g] = (uint32_t)min(r, M - 1 - m0) * ldxb + (((lane & 7) ^ ((r >> 1) & 7)) * 16);  // rows past M repeat the last one, never stored
  }
  const bool pair = kind == EPI_SWIGLU || kind == EPI_QKV || (kind == kEpiPart && P.kind == EPI_QKV);
  // 8 tile columns c .. c + 7 lie in one half of one wave's 32 TJ columns; pair epilogues
  // keep the even columns in the first half and their odd partners in the second, so a
  // lane holds both values of its pairs.  wbase: the matrix (of the tile, or of the half)
  // and its first row; step: rows between columns.
  const bool gu = kind == EPI_SWIGLU;
  const int which = kind == EPI_QKV || (kind == kEpiPart && P.mats.mode == MAT_QKV) ? (bx >= P.cm) + (bx >= 2 * P.cm) : 0;  // a tile lies in one of q, k, v
  const char* const wm0 = reinterpret_cast<const char*>(which == 0 ? P.mats.m[0] : which == 1 ? P.mats.m[1] : P.mats.m[2]);
  const char* const wm1 = reinterpret_cast<const char*>(gu ? P.mats.m[1] : wm0);
  // the tile's first column in its matrix, and in the fused order.  A matrix of an odd
  // multiple of 64 rows ends inside its last 128 tile, on a wave boundary: that tile's
  // second wave column repeats the first one's weights and stores nothing (a forward of
  // 2048 rows, on 64 x 64 tiles without this: d = 960 2.36 -> 1.74 ms, d = 1600 5.48 -> 3.24).
  const int ncol = (bx - which * P.cm) * BN, n0 = ncol + which * P.mats.rows, nrow = gu ? ncol >> 1 : ncol;
  const int wcols = WN == 2 && WM == 2 && !gu && ncol + 32 * TJ >= P.mats.rows ? 1 : WN;  // wave columns inside the matrix
  const uint32_t vrow = (uint32_t)(lane >> 3) * (uint32_t)(pair && !gu ? 2 : 1) * (uint32_t)K * 2;
#pragma unroll
  for (int g = 0; g < GB; ++g) {
    const int c = (wave * GB + g) * 8, cc = c % (32 * TJ), odd = cc / (16 * TJ), in = cc % (16 * TJ), wc = min(c / (32 * TJ), wcols - 1);
    const int r = gu ? nrow + wc * 16 * TJ + in : nrow + wc * 32 * TJ + (pair ? 2 * in + odd : cc);
    sb[g] = (pair && odd ? wm1 : wm0) + ((size_t)r * K + kz * 32) * 2;
    vb[g] = vrow + (((lane & 7) ^ (((c + (lane >> 3)) >> 1) & 7)) * 16);
  }
  const int wm = wave / WN, wn = wave % WN;
  const char* sx = reinterpret_cast<const char*>(P.x) + (size_t)m0 * ldxb + kz * 128;
  const uint32_t lbase = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
  // piece g of step k's X into the slot at buf, of weight step j (two steps) into slot j % 2
  auto req_a = [&](int g, int k, uint32_t buf) __attribute__((always_inline)) {
    // past the end: the last step again, unused
    dma16(lbase + buf + (uint32_t)(wave * GA + g) * 1024, va[g], sx + (size_t)min(k, nk - 1) * 128);
  };
  auto req_w = [&](int g, int j) __attribute__((always_inline)) {
    dma16(lbase + 3 * T::kA + (uint32_t)(j & 1) * T::kW + (uint32_t)(wave * GB + g) * 1024, vb[g],
          sb[g] + (size_t)min(j, nk / 2 - 1) * 128);
  };
  f32x16 acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  struct Frag {
    bf16x8 h[TI], l[TI], w[TJ];
  };
  // lane's row and 16-byte chunk of a fragment: chunk 2 ks + lane / 32 (+ 4: lo half, or
  // the odd step of a weight slot), XOR-ed as stored
  const int frow = lane & 31, fsw = (lane >> 1) & 7;
  const char* const pa = lds + (wm * 32 * TI + frow) * 128;
  const char* const pb = lds + 3 * T::kA + (wn * 32 * TJ + frow) * 128;
  const uint32_t ch[4] = {(uint32_t)((0 + (lane >> 5)) ^ fsw) * 16, (uint32_t)((2 + (lane >> 5)) ^ fsw) * 16,
                          (uint32_t)((4 + (lane >> 5)) ^ fsw) * 16, (uint32_t)((6 + (lane >> 5)) ^ fsw) * 16};
  // fragment i of half ks of a step: weights (slot wbuf, odd step of the slot or even),
  // then the hi and lo halves of X (slot abuf)
  auto read1 = [&](Frag& f, int i, uint32_t abuf, uint32_t wbuf, int odd, int ks) __attribute__((always_inline)) {
    if (i < TJ) f.w[i] = *reinterpret_cast<const bf16x8*>(pb + wbuf + ch[2 * odd + ks] + i * 4096);
    else if (i < TJ + TI) f.h[i - TJ] = *reinterpret_cast<const bf16x8*>(pa + abuf + ch[ks] + (i - TJ) * 4096);
    else f.l[i - TJ - TI] = *reinterpret_cast<const bf16x8*>(pa + abuf + ch[2 + ks] + (i - TJ - TI) * 4096);
  };
  constexpr int kReads = TJ + 2 * TI, kMma = 2 * TI * TJ;
  // The half step's MFMAs on f, with the reads of the next half step into g and up to NQ
  // loads of later steps between them: issued in a bunch, they hold the wave's next
  // MFMA back until the LDS and memory queues have taken them.
  auto half_step = [&](const Frag& f, Frag& g, uint32_t abuf, uint32_t wbuf, auto odd, auto ks, auto nq, auto&& load) __attribute__((always_inline)) {
    static_for<kMma>([&](auto mc) __attribute__((always_inline)) {
      constexpr int m = decltype(mc)::value, lo = m / (TI * TJ), i = m % (TI * TJ) / TJ, j = m % TJ, NQ = decltype(nq)::value;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo ? f.l[i] : f.h[i], f.w[j], acc[i][j], 0, 0, 0);
      constexpr int r0 = m * kReads / kMma, r1 = (m + 1) * kReads / kMma;
      if constexpr (r1 > r0) read1(g, r0, abuf, wbuf, decltype(odd)::value, decltype(ks)::value);
      constexpr int q0 = m * NQ / kMma, q1 = (m + 1) * NQ / kMma;
      if constexpr (q1 > q0) load(q0);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  using C4 = std::integral_constant<int, 4>;
  using C8 = std::integral_constant<int, 8>;
#pragma unroll
  for (int g = 0; g < GB; ++g) req_w(g, 0);
#pragma unroll
  for (int g = 0; g < GA; ++g) req_a(g, 0, 0);
#pragma unroll
  for (int g = 0; g < GA; ++g) req_a(g, 1, T::kA);
#pragma unroll
  for (int g = 0; g < GB; ++g) req_w(g, 1);
#pragma unroll
  for (int g = 0; g < GA; ++g) req_a(g, 2, 2 * T::kA);
  asm volatile("s_waitcnt vmcnt(12)\n\ts_barrier" ::"s"(lbase) : "memory");
  // lane l holds the scale of row l of the wave's 64 (bytes of x, unused, when not scaled);
  // one more load in flight only makes the first step's wait stricter
  static_assert(TI == 2, "64 rows per wave");
  const float rsl = kind != EPI_RESID ? P.rs[min(m0 + wm * 64 + lane, M - 1)] : 0.f;
  Frag f0, f1;
  uint32_t a0 = 0, a1 = T::kA, a2 = 2 * T::kA;  // slots of steps k, k + 1, k + 2
#pragma unroll
  for (int i = 0; i < kReads; ++i) read1(f0, i, 0, 0, 0, 0);
  // Step k: the second half's fragments are read during the first half's MFMAs.  Then
  // every wave has read the whole step, so behind the barrier its X slot takes step
  // k + 3 and, after an odd step, its weight slot those of steps k + 3 and k + 4; the
  // next step's first fragments are read during the second half's MFMAs.  What a step
  // needs is waited for at the barrier before it, and was requested behind the barrier
  // two steps earlier: an even step's barrier leaves the 8 loads requested in the step
  // before it (weights, then X) in flight, an odd one's 4.
  uint32_t w = 0;
  for (int k = 0; k < nk; k += 2) {
    half_step(f0, f1, a0, w, C0(), C1(), C0(), [](int) {});
    asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    half_step(f1, f0, a1, w, C1(), C0(), C4(), [&](int q) __attribute__((always_inline)) { req_a(q, k + 3, a0); });
    half_step(f0, f1, a1, w, C1(), C1(), C0(), [](int) {});
    asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    half_step(f1, f0, a2, T::kW - w, C0(), C0(), C8(), [&](int q) __attribute__((always_inline)) {
      if (q < GB) req_w(q, k / 2 + 2);
      else req_a(q - GB, k + 4, a1);
    });
    const uint32_t t = a0;
    a0 = a2;
    a2 = a1;
    a1 = t;
    w = T::kW - w;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load may land after the block has ended
  if (wn >= wcols) return;
  // The epilogue's row and column numbers start here: computed from the same values as the
  // loop's, the compiler would move them above the loop and spill.
  int em = m0 + wm * 32 * TI, en = n0, el = lane, ew = wn, ec = nrow;
  asm volatile("" : "+s"(em), "+s"(en), "+v"(el), "+s"(ew), "+s"(ec));
  const int jj = el & 31, half = el >> 5;
  const bool full = m0 + BM <= M;
  auto row_of = [&](int i, int r) { return em + i * 32 + 8 * (r >> 2) + 4 * half + (r & 3); };
  if (kind != EPI_RESID && P.scaled) {
    static_for<TI>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float sc = __shfl(rsl, i * 32 + 8 * (r >> 2) + 4 * half + (r & 3));
        static_for<TJ>([&](auto jc) __attribute__((always_inline)) { acc[i][decltype(jc)::value][r] *= sc; });
      }
    });
  }
  if (kind == kEpiPart) {
    // sums of this K range, columns in the matrix's order: gemm_finish_kernel adds
    // the ranges and runs the epilogue
    float* part = P.part + (size_t)blockIdx.z * M * P.N;
    static_for<TI>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = row_of(i, r);
        if (full || m < M) {
          float* y = part + (size_t)m * P.N + en + ew * 32 * TJ;
          if (pair) {
            static_for<TJ / 2>([&](auto jc) __attribute__((always_inline)) {
              constexpr int j = decltype(jc)::value;
              *reinterpret_cast<float2*>(y + 2 * (j * 32 + jj)) = make_float2(acc[i][j][r], acc[i][j + TJ / 2][r]);
            });
          } else {
            static_for<TJ>([&](auto jc) __attribute__((always_inline)) {
              constexpr int j = decltype(jc)::value;
              y[j * 32 + jj] = acc[i][j][r];
            });
          }
        }
      }
    });
  } else if (kind == EPI_SWIGLU) {
    // silu(gate) * up as split rows; neighbouring lanes trade values so that each stores two
    // columns of one row as one word: the even lane row r, the odd one row r + 1
    const size_t ldy = (size_t)P.ldy * 2;
    // Short passes (the 128 tile) keep the division form's accuracy; the 256 tile's long
    // ones take the bare hardware exp2 and reciprocal.  Products of an M = 600 forward, d =
    // 1024, 13 layers: bare 1225 us, silu_near 1234, division 1247.
    auto act = [](float x) { return T::NW == 8 ? silu_fast(x) : silu_near(x); };
    static_for<TI>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        const int m = row_of(i, r) + (jj & 1);
        static_for<TJ / 2>([&](auto jc) __attribute__((always_inline)) {
          constexpr int j = decltype(jc)::value;
          const float v0 = act(acc[i][j][r]) * acc[i][j + TJ / 2][r];
          const float v1 = act(acc[i][j][r + 1]) * acc[i][j + TJ / 2][r + 1];
          const float got = dpp<kDppXor1>((jj & 1) ? v0 : v1);
          const float c0 = (jj & 1) ? got : v0, c1 = (jj & 1) ? v1 : got;
          uint32_t hi, lo;
          bf16_hi_lo2(c0, c1, hi, lo);
          // 32 columns' group of the split row: hi halves, then lo
          uint16_t* y = P.y + (size_t)m * ldy + 2 * ((en >> 1) + ew * 16 * TJ + j * 32) + (jj & ~1);
          if (full || m < M) {
            *reinterpret_cast<uint32_t*>(y) = hi;
            *reinterpret_cast<uint32_t*>(y + 32) = lo;
          }
        });
      }
    });
  } else if (kind == EPI_QKV) {
    const Epi e = P.epi;
    const int col0 = ec + ew * 32 * TJ;
    static_for<TI>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = row_of(i, r);
        const int mc = min(m, M - 1);
        const int pos = which < 2 ? e.tok.pos[mc] : 0;
        size_t crow = 0;
        if (which > 0) crow = (size_t)e.tok.b[mc] * e.b_stride + (size_t)e.tok.slot[mc] * e.dh;
        static_for<TJ / 2>([&](auto jc) __attribute__((always_inline)) {
          constexpr int j = decltype(jc)::value;
          const int c = col0 + 2 * (j * 32 + jj);
          const int h = e.dh == 64 ? c >> 6 : c >> 5, ee = c & (e.dh - 1);
          float a0 = acc[i][j][r], a1 = acc[i][j + TJ / 2][r];
          if (which < 2) {
            const float2 cs = e.rope[(size_t)pos * (e.dh >> 1) + (ee >> 1)];
            const float r0 = a0 * cs.x - a1 * cs.y, r1 = a0 * cs.y + a1 * cs.x;
            a0 = r0;
            a1 = r1;
          }
          if (full || m < M) {
            if (which == 0) {
              *reinterpret_cast<float2*>(e.Q + (size_t)m * e.d + c) = make_float2(a0, a1);
            } else {
              char* cache = reinterpret_cast<char*>(which == 1 ? e.kc : e.vc);
              const size_t off = crow + (size_t)h * e.cap * e.dh + ee;
              if (e.kvt == 2) {
                const uint32_t u0 = __builtin_bit_cast(uint16_t, (_Float16)fminf(fmaxf(a0, -65504.0f), 65504.0f));
                const uint32_t u1 = __builtin_bit_cast(uint16_t, (_Float16)fminf(fmaxf(a1, -65504.0f), 65504.0f));
                *reinterpret_cast<uint32_t*>(cache + off * 2) = u0 | (u1 << 16);
              } else if (e.kvt == 1) {
                *reinterpret_cast<uint32_t*>(cache + off * 2) = (uint32_t)f2bf(a0) | ((uint32_t)f2bf(a1) << 16);
              } else {
                *reinterpret_cast<float2*>(cache + off * 4) = make_float2(a0, a1);
              }
            }
          }
        });
      }
    });
  } else {
    float* const Y = P.epi.Y;
    const size_t ldy = (size_t)P.epi.ldy;
    static_for<TI>([&](auto ic) __attribute__((always_inline)) {
      constexpr int i = decltype(ic)::value;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = row_of(i, r);
        float* y = Y + (size_t)m * ldy + en + ew * 32 * TJ + jj;
        if (full || m < M) {
          float old[TJ];
#pragma unroll
          for (int j = 0; j < TJ; ++j) old[j] = y[j * 32];
          static_for<TJ>([&](auto jc) __attribute__((always_inline)) {
            constexpr int j = decltype(jc)::value;
            y[j * 32] = old[j] + acc[i][j][r];
          });
        }
      }
    });
  }
}

// Split rows of float32 rows: x, or x * gain and rs = 1 / RMS(x); a wave per row.  Eight lanes read
// a group's 128 bytes in one load and write them back as its halves, so y may be x.
// V > 0: rows of d = 256 V values, all of whose loads are in flight at once (the split,
// copy and norm kernels of a forward of 4096 rows, general loop -> this: d = 1024 161 ->
// 154 us, d = 2048 284 -> 254; 16384 rows 465 -> 435, 950 -> 885; nothing at 256 rows).
template <int V>
__global__ __launch_bounds__(256) void split_rows_kernel(const float* x, const float* gain, float eps, uint16_t* y, float* rs,
                                                         int d, int M) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= M) return;
  const float* xr = x + (size_t)row * d;
  uint16_t* yr = y + (size_t)row * 2 * d;
  auto put = [&](float4 t, int k) {
    if (gain != nullptr) {
      const float4 g = *reinterpret_cast<const float4*>(gain + k);
      t.x *= g.x; t.y *= g.y; t.z *= g.z; t.w *= g.w;
    }
    uint32_t h0, l0, h1, l1;
    bf16_hi_lo2(t.x, t.y, h0, l0);
    bf16_hi_lo2(t.z, t.w, h1, l1);
    uint16_t* o = yr + 2 * (k & ~31) + (k & 31);
    *reinterpret_cast<uint2*>(o) = make_uint2(h0, h1);
    *reinterpret_cast<uint2*>(o + 32) = make_uint2(l0, l1);
  };
  auto sq = [](float4 t) { return t.x * t.x + t.y * t.y + t.z * t.z + t.w * t.w; };
  float ss = 0.f;
  if constexpr (V > 0) {
    float4 v[V];
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = *reinterpret_cast<const float4*>(xr + i * 256 + lane * 4);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      ss += sq(v[i]);
      put(v[i], i * 256 + lane * 4);
    }
  } else {
    for (int k = lane * 4; k < d; k += 256) {
      const float4 t = *reinterpret_cast<const float4*>(xr + k);
      ss += sq(t);
      put(t, k);
    }
  }
  if (gain != nullptr) {
    ss = wave_sum(ss);
    if (lane == 0) rs[row] = 1.0f / sqrtf(ss / (float)d + eps);
  }
}

// The second half of a split-K product onto the residual rows and the split before the
// next linear in one pass: row m of x gets the sum of its ks partial rows (added in order
// z = 0, 1, ..., then to x, as gemm_finish_kernel does), y the split row of x * gain and
// rs its 1 / RMS.  A block per row; bound by its launch and one round of loads (at
// 531 rows the two kernels it replaces took 5.5 + 5.4 us).
__global__ __launch_bounds__(256) void finish_split_kernel(const float* part, int ks, int M, int d, float* x, const float* gain,
                                                           float eps, uint16_t* y, float* rs) {
  __shared__ float red[4];
  const int row = blockIdx.x, tid = threadIdx.x;
  const size_t zs = (size_t)M * d;
  float ss = 0.f;
  for (int k = tid * 4; k < d; k += 1024) {
    const float4 old = *reinterpret_cast<const float4*>(x + (size_t)row * d + k);
    const float4 g = *reinterpret_cast<const float4*>(gain + k);
    const float* pp = part + (size_t)row * d + k;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
    for (int z = 0; z < ks; ++z) {
      const float4 t = *reinterpret_cast<const float4*>(pp + z * zs);
      a.x += t.x; a.y += t.y; a.z += t.z; a.w += t.w;
    }
    a.x += old.x; a.y += old.y; a.z += old.z; a.w += old.w;
    *reinterpret_cast<float4*>(x + (size_t)row * d + k) = a;
    ss += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
    uint32_t h0, l0, h1, l1;
    bf16_hi_lo2(a.x * g.x, a.y * g.y, h0, l0);
    bf16_hi_lo2(a.z * g.z, a.w * g.w, h1, l1);
    uint16_t* o = y + (size_t)row * 2 * d + 2 * (k & ~31) + (k & 31);
    *reinterpret_cast<uint2*>(o) = make_uint2(h0, h1);
    *reinterpret_cast<uint2*>(o + 32) = make_uint2(l0, l1);
  }
  ss = wave_sum(ss);
  if ((tid & 63) == 0) red[tid >> 6] = ss;
  __syncthreads();
  if (tid == 0) rs[row] = 1.0f / sqrtf((red[0] + red[1] + red[2] + red[3]) / (float)d + eps);
}

// Column blocks of BN: a tile lies in one matrix of a fused QKV weight.
int column_blocks(const PlaneLinear& P, int BN) {
  return P.mats.mode == MAT_QKV ? 3 * ((P.mats.rows + BN - 1) / BN) : (P.N + BN - 1) / BN;
}

template <int WM, int WN, int TI, int TJ>
hipError_t planes_launch_t(PTile<WM, WN, TI, TJ>, const PlaneLinear& P, int ks, hipStream_t st, const Ev& ev) {
  using T = PTile<WM, WN, TI, TJ>;
  PlaneLinear Q = P;
  Q.ksplit = ks;
  Q.scaled = P.rs != nullptr;
  if (!Q.scaled) Q.rs = reinterpret_cast<const float*>(P.x);  // M readable floats
  Q.cm = (P.mats.rows + T::BN - 1) / T::BN;
  Q.cb = column_blocks(P, T::BN);
  const int rb = (P.M + T::BM - 1) / T::BM;
  // row blocks per L2 group: about 2 MiB of activation rows, a power of two; the kernel
  // divides an XCD's block number by the group's blocks with a rounded-up reciprocal, exact
  // while the product of the two is below 2^32
  int grl = 0;
  while (grl < 3 && ((int64_t)T::BM * P.K * 4 << (grl + 1)) <= (2 << 20)) ++grl;
  const int64_t group = (int64_t)Q.cb << grl;
  Q.grl = grl;
  Q.ginv = 0;
  if (ks == 1 && rb % (8 << grl) == 0 && group > 1 && (int64_t)rb * Q.cb / 8 * group < ((int64_t)1 << 32))
    Q.ginv = (uint32_t)((((uint64_t)1 << 32) + group - 1) / group);
  auto go = [&](auto kern) {
    return plaunch(kern, dim3(Q.cb, rb, ks), dim3(64 * T::NW), st, ev.start, ks > 1 ? nullptr : ev.stop, Q);
  };
  if constexpr (T::NW == 8) {
    if (ks > 1) return hipErrorInvalidValue;  // the 256 tile is not split
    return go(gemm_planes_kernel<WM, WN, TI, TJ, kEpiAny>);
  } else {
    if (ks > 1) return go(gemm_planes_kernel<WM, WN, TI, TJ, kEpiPart>);
    switch (P.kind) {
      case EPI_SWIGLU: return go(gemm_planes_kernel<WM, WN, TI, TJ, EPI_SWIGLU>);
      case EPI_QKV: return go(gemm_planes_kernel<WM, WN, TI, TJ, EPI_QKV>);
      case EPI_RESID: return go(gemm_planes_kernel<WM, WN, TI, TJ, EPI_RESID>);
      default: return hipErrorInvalidValue;
    }
  }
}

}  // namespace

bool planes_fit(int M, int N, int K, int n_mat) {
  return M >= kPlanesMinRows && N % 64 == 0 && n_mat % 64 == 0 && K % 64 == 0 && K >= 128;
}

// The 256 tile fills the chip with one block per compute unit, the 128 tile with two; a
// round of the chip on 128 tiles takes about 0.54 of one on 256 tiles, and 0.40 when at
// most one block per unit is left for it (gate/up, K = 1024: M = 2048 in one round of
// 256 tiles 53 us, two of 128 tiles 59 us; M = 4096, N = 3072: 76 us in three quarters
// of a round of 256 tiles, 68 us in one and a half of 128).  A grid of few 128 tiles
// splits K: once up to 200 tiles (M = 740, N = 3072, K = 1024: 31 -> 27 us), again while
// the blocks stay below 200 (M = 740, N = 1024, K = 4096: 48 us whole, 30 / 27 / 29 us
// in 2 / 4 / 8 parts; M = 512: 48, 28 / 21 / 24 us), a part keeping 256 columns.
PlanesPlan planes_plan(const PlaneLinear& P) {
  const int64_t t128 = (int64_t)column_blocks(P, 128) * ((P.M + 127) / 128);
  const int nmat = P.mats.mode == MAT_QKV ? P.mats.rows : P.N;
  // gate/up of K > 4096 keeps the 128 tile, whose silu is the nearer one
  if (P.N % 256 == 0 && nmat % 256 == 0 && !(P.kind == EPI_SWIGLU && P.K > 4096)) {
    const int64_t t256 = (int64_t)(P.N / 256) * ((P.M + 255) / 256);
    const int64_t rem = t128 % 512;
    if (100 * ((t256 + 255) / 256) <= 54 * (t128 / 512) + (rem == 0 ? 0 : rem <= 256 ? 40 : 54)) return {256, 1};
  }
  int ks = 1;
  if (P.kind != EPI_SWIGLU && P.part != nullptr)
    while (t128 * ks * 2 <= (ks == 1 ? 400 : 200) && P.K % (64 * 2 * ks) == 0 && P.K / (2 * ks) >= 256 &&
           (int64_t)ks * 2 * P.M * P.N <= kGemmPartFloats)
      ks *= 2;
  return {128, ks};
}

namespace {
// K splits of a residual product (d columns) of M rows over K.
int resid_ks(int M, int d, int K) {
  PlaneLinear P{};
  float part;  // the rule only asks whether there is scratch
  P.kind = EPI_RESID; P.M = M; P.N = d; P.K = K; P.part = &part;
  P.mats.rows = d; P.mats.mode = MAT_SINGLE;
  return planes_plan(P).ks;
}
}  // namespace

// Split rows against the tiles of kernels.hip, us per layer of a prompt pass (off -> on):
// a layer whose residual products split K norms their rows in the kernel that adds the
// parts, so it takes no launch more, and the line lies where 128-row tiles are filled
// (d = 1024: M = 65 78.3 -> 80.1, 96 81.9 -> 81.9, 128 91.8 -> 85.4; d = 768: M = 128
// 76.5 -> 79.5, 192 84.3 -> 83.3; d = 2048: M = 65 139 -> 122).  The others split their
// rows in two launches of their own and walk K whole, which long passes repay (d = 128:
// M = 512 65.9 -> 79.9, 8192 128 -> 127, 32768 304 -> 270; d = 256: M = 1024 89 -> 109,
// 4096 133 -> 128; d = 384: 2048 148 -> 146; d = 576: 512 99 -> 115, 1024 142 -> 138;
// d = 960: 256 106 -> 131, 512 152 -> 144; d = 1600: 128 128 -> 171, 256 189 -> 175).
// Both lines follow M d sqrt(d_ff) over these widths.
bool planes_layer(int M, int d, int d_ff) {
  if (!planes_fit(M, 3 * d, d, d) || !planes_fit(M, d, d, d) || !planes_fit(M, 2 * d_ff, d, 2 * d_ff) || !planes_fit(M, d, d_ff, d))
    return false;
  const double work = (double)M * d * sqrt((double)d_ff);
  return work >= (resid_ks(M, d, d) > 1 && resid_ks(M, d, d_ff) > 1 ? 6e6 : 3.2e7);
}

// One MLP head (gate/up and down, no residual rows to norm before them), off -> on: d =
// 512 M = 128 75 -> 72, 512 140 -> 142; d = 1024: 65 82.5 -> 82.8, 256 114 -> 108; d =
// 2048: 65 148 -> 138; d = 128 and 256: 65 +3, 512 no difference.
bool planes_head(int M, int d, int d_ff) {
  return planes_fit(M, 2 * d_ff, d, 2 * d_ff) && planes_fit(M, d, d_ff, d) && (double)M * d * sqrt((double)d_ff) >= 1.2e7;
}

static bool fuse_shape(const PlaneLinear& P) { return P.kind == EPI_RESID && P.epi.ldy == P.N; }

bool planes_fuses_norm(const PlaneLinear& P) { return fuse_shape(P) && planes_plan(P).ks > 1; }

hipError_t launch_planes_at(const PlaneLinear& P, PlanesPlan plan, hipStream_t st, const Ev& ev) {
  const hipError_t e = plan.tile == 256 ? planes_launch_t(PTile256{}, P, plan.ks, st, ev) : planes_launch_t(PTile128{}, P, plan.ks, st, ev);
  if (e != hipSuccess || plan.ks == 1) return e;
  if (P.next != nullptr && fuse_shape(P))
    return plaunch(finish_split_kernel, dim3(P.M), dim3(256), st, nullptr, ev.stop, (const float*)P.part, plan.ks, P.M, P.N,
                   P.epi.Y, P.next_gain, P.eps, P.next, P.next_rs);
  Linear L{};
  L.M = P.M; L.K = P.K; L.N = P.N; L.epi = P.epi; L.epi.kind = P.kind; L.part = P.part;
  return launch_gemm_finish(L, plan.ks, st, ev);
}

hipError_t launch_planes(const PlaneLinear& P, hipStream_t st, const Ev& ev) {
  if (P.M <= 0) return hipSuccess;
  return launch_planes_at(P, planes_plan(P), st, ev);
}

hipError_t launch_split_rows(const float* x, const float* gain, float eps, uint16_t* y, float* rs, int d, int M,
                             hipStream_t st, const Ev& ev) {
  if (M <= 0) return hipSuccess;
  const dim3 grid((M + 3) / 4);
  auto go = [&](auto kern) { return plaunch(kern, grid, dim3(256), st, ev.start, ev.stop, x, gain, eps, y, rs, d, M); };
  if (d == 1024) return go(split_rows_kernel<4>);
  if (d == 2048) return go(split_rows_kernel<8>);
  return go(split_rows_kernel<0>);
}

}  // namespace mbp

// For the tests: whether the linears of a block (head = 0) or of an MLP head (1) of M rows
// run on split rows.
extern "C" int mbp_check_split_layer(int32_t M, int32_t d, int32_t d_ff, int32_t head) {
  return head ? mbp::planes_head(M, d, d_ff) : mbp::planes_layer(M, d, d_ff);
}

// For the tests: one product on split rows at a given tile and K splits (tile 0: the plan's
// own), from float32 rows, on the default stream; caches hold float32, all rows are batch
// row 0.  1: refused.
struct MbpCheckProduct {
  int32_t kind, tile, ks, M, N, K, rows, dh, cap;
  float eps;
  const float *x, *gain;
  uint16_t* xs;  // [M, 2 K] split rows of x (* gain)
  float* rs;     // [M]
  const void* w[3];
  uint16_t* ys;  // SWIGLU: [M, N] (2 x N / 2)
  float* y;      // RESID: [M, N]; QKV: Q [M, rows]
  float* part;
  const int32_t *zero, *pos, *slot;
  const float* rope;
  void *kc, *vc;  // [rows / dh, cap, dh]
  uint16_t* next;
  const float* next_gain;
  float* next_rs;
};

extern "C" int mbp_check_product(const MbpCheckProduct* c) {
  using namespace mbp;
  PlaneLinear P{};
  P.x = c->xs; P.rs = c->gain != nullptr ? c->rs : nullptr; P.ldx = c->K; P.M = c->M; P.K = c->K; P.N = c->N; P.kind = c->kind;
  for (int i = 0; i < 3; ++i) P.mats.m[i] = c->w[i];
  P.mats.rows = c->rows;
  P.mats.mode = c->kind == EPI_QKV ? MAT_QKV : c->kind == EPI_SWIGLU ? MAT_GATEUP : MAT_SINGLE;
  P.y = c->ys; P.ldy = c->N / 2; P.part = c->part;
  P.epi.kind = c->kind; P.epi.Y = c->y; P.epi.ldy = c->N; P.epi.Q = c->y; P.epi.kc = c->kc; P.epi.vc = c->vc;
  P.epi.cap = c->cap; P.epi.dh = c->dh; P.epi.H = c->dh > 0 ? c->rows / c->dh : 0; P.epi.d = c->rows;
  P.epi.rope = reinterpret_cast<const float2*>(c->rope);
  P.epi.tok.b = c->zero; P.epi.tok.pos = c->pos; P.epi.tok.slot = c->slot; P.epi.tok.M = c->M;
  P.next = c->next; P.next_gain = c->next_gain; P.eps = c->eps; P.next_rs = c->next_rs;
  const bool whole = c->kind == EPI_QKV ? c->N == 3 * c->rows : c->kind == EPI_SWIGLU ? c->N == 2 * c->rows : c->kind == EPI_RESID && c->N == c->rows;
  if (c->M < 1 || !whole || c->N % 64 || c->rows % 64 || c->K % 64 || c->K < 128) return 1;
  const PlanesPlan plan = c->tile == 0 ? planes_plan(P) : PlanesPlan{c->tile, c->ks};
  if (plan.tile != 128 && (plan.tile != 256 || plan.ks != 1 || c->N % 256 || (c->kind == EPI_QKV ? c->rows : c->N) % 256)) return 1;
  if (plan.ks < 1 || c->K % (64 * plan.ks) || c->K / plan.ks < 128) return 1;
  if (plan.ks > 1 && (c->kind == EPI_SWIGLU || c->part == nullptr || (int64_t)plan.ks * c->M * c->N > kGemmPartFloats)) return 1;
  hipError_t e = launch_split_rows(c->x, c->gain, c->eps, c->xs, c->rs, c->K, c->M, nullptr);
  if (e == hipSuccess) e = launch_planes_at(P, plan, nullptr);
  if (e == hipSuccess) e = hipStreamSynchronize(nullptr);
  return e == hipSuccess ? 0 : 2;
}
