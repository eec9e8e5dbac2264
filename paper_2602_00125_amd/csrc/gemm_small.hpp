// Matrix-core GEMM for products too small to fill the chip with ring tiles
// (gemm_dma.hpp), gfx950 only: few rows, few columns, or both.
//
// Such a product is bound by latency: by the serial chain of K-stages of a
// block and by how few blocks there are. So a block computes one small tile
// (64x64, 32x32 or 16x16) and its waves share the contraction instead of the
// tile: wave w multiplies its run of K-steps for the whole tile, with
// operands loaded from global memory straight into fragment registers, several
// K-steps ahead (no LDS, no barrier in the loop), and the waves' partial tiles
// meet in LDS at the end, where they are added in wave order on the way to C.
// Loads need no alignment beyond the element's and no padded copies: rows past
// the matrix are read from the last row (their results are dropped), the K
// tail element by element. A wave whose sums are not finite (what the split
// of fp32 values does not serve) takes its share again by the fp32 instructions.
//
// v_mfma_f32_16x16x32_bf16: lane l of the first (second) operand holds row
// (column) l & 15, k group g = l >> 4. A K-step is 32 k, dealt to the groups by
// small_k on both operands. fp32 values are split in three bf16 parts, six
// products a pair, scaled as in DmaMma<float>. An operand contiguous along m (n) instead is read T
// consecutive rows at a time (T tiles): tile i's row r is row T r + i.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "act.hpp"
#include "gemm_dma.hpp"
#include "gemm_kernel.hpp"
#include "gemm_params.hpp"

namespace mt {
namespace gemm {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

template <typename T>
struct SmallOperand;

// Raw fp32 values of T tiles over a K-step, and the MFMA operands made of them.
template <>
struct SmallOperand<float> {
  using Elem = float;
  struct Raw {
    float x[8];
  };
  struct Frag {
    bf16x8 h, m, l;
  };
  static __device__ __forceinline__ void set(Raw& r, int e, float v) { r.x[e] = v; }
  static __device__ __forceinline__ Frag frag(const Raw& r, float scale) {
    uint32_t c0 = 0x0000bf80u, c1 = 0xbf800000u;  // (-1, 0), (0, -1): see DmaMma<float>::split
    __asm__("" : "+s"(c0), "+s"(c1));
    const bf16x2 n0 = __builtin_bit_cast(bf16x2, c0), n1 = __builtin_bit_cast(bf16x2, c1);
    u32x4 h, m, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const f32x2 v = {r.x[2 * e] * scale, r.x[2 * e + 1] * scale};
      const bf16x2 hh = __builtin_convertvector(v, bf16x2);
      const f32x2 s = {__builtin_amdgcn_fdot2_f32_bf16(hh, n0, v[0], false),
                       __builtin_amdgcn_fdot2_f32_bf16(hh, n1, v[1], false)};
      const bf16x2 mm = __builtin_convertvector(s, bf16x2);
      const f32x2 q = {__builtin_amdgcn_fdot2_f32_bf16(mm, n0, s[0], false),
                       __builtin_amdgcn_fdot2_f32_bf16(mm, n1, s[1], false)};
      h[e] = __builtin_bit_cast(uint32_t, hh);
      m[e] = __builtin_bit_cast(uint32_t, mm);
      l[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(q, bf16x2));
    }
    return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
  }
  template <int TN>
  static __device__ __forceinline__ void mfma(const Frag& a, const Frag (&b)[TN], f32x4 (&acc)[TN]) {
    auto step = [&](bf16x8 Frag::*pb, bf16x8 Frag::*pa) {
#pragma unroll
      for (int q = 0; q < TN; ++q)
        acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[q].*pb, a.*pa, acc[q], 0, 0, 0);
    };
    step(&Frag::l, &Frag::h);
    step(&Frag::h, &Frag::l);
    step(&Frag::m, &Frag::m);
    step(&Frag::m, &Frag::h);
    step(&Frag::h, &Frag::m);
    step(&Frag::h, &Frag::h);
  }
  // by the fp32 instructions: element e of every group is one k of four
  template <int TN>
  static __device__ __forceinline__ void plain(const Raw& a, const Raw (&b)[TN], f32x4 (&acc)[TN]) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int q = 0; q < TN; ++q) acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[q].x[e], a.x[e], acc[q], 0, 0, 0);
  }
  static __device__ __forceinline__ float sum(const Raw& r) {
    return ((r.x[0] + r.x[1]) + (r.x[2] + r.x[3])) + ((r.x[4] + r.x[5]) + (r.x[6] + r.x[7]));
  }
  static constexpr bool SPLIT = true;
  static constexpr float UNSCALE = X6_UNSCALE;  // of the accumulators
};

template <>
struct SmallOperand<__bf16> {
  using Elem = unsigned short;
  struct Raw {
    u16x8 x;
  };
  struct Frag {
    bf16x8 v;
  };
  static __device__ __forceinline__ void set(Raw& r, int e, unsigned short v) { r.x[e] = v; }
  static __device__ __forceinline__ Frag frag(const Raw& r, float) { return {__builtin_bit_cast(bf16x8, r.x)}; }
  template <int TN>
  static __device__ __forceinline__ void mfma(const Frag& a, const Frag (&b)[TN], f32x4 (&acc)[TN]) {
#pragma unroll
    for (int q = 0; q < TN; ++q)
      acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[q].v, a.v, acc[q], 0, 0, 0);
  }
  static constexpr bool SPLIT = false;
  static constexpr float UNSCALE = 1.f;
  static __device__ __forceinline__ float value(unsigned short v) { return __uint_as_float((uint32_t)v << 16); }
  static __device__ __forceinline__ float sum(const Raw& r) {
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) s += value(r.x[e]);
    return s;
  }
};

// k of element e of group g within a K-step: 4 g + e and 16 + 4 g + e - 4
// (fp32) or 8 g + e (bf16), so that a lane's 16-byte loads of a K-contiguous
// row and its three neighbours' are 64 consecutive bytes
template <typename T>
__device__ __forceinline__ int small_k(int g, int e) {
  return sizeof(T) == 4 ? 4 * g + (e & 3) + 16 * (e >> 2) : 8 * g + e;
}

// One operand of the wave's tile: NT tiles of 16 rows (columns for B).
template <typename T, bool KC, int NT>
struct SmallLoader {
  using Op = SmallOperand<T>;
  using E = typename Op::Elem;
  typedef E ev4 __attribute__((ext_vector_type(4), aligned(sizeof(E))));
  typedef unsigned short ev8 __attribute__((ext_vector_type(8), aligned(2)));
  typedef E evn __attribute__((ext_vector_type(NT == 1 ? 2 : NT), aligned(sizeof(E))));
  static constexpr int ES = (int)sizeof(E);
  const E* base;   // element (first row of the tile, k = 0) of this batch element
  int64_t ld;
  int64_t left;    // rows from the tile's first to the matrix's end
  uint32_t off[KC ? NT : 1];  // bytes from the K-step's origin (the host bounds ld)

  __device__ __forceinline__ void init(const void* p, int64_t off0, int64_t r0, int64_t ld_, int64_t rows, int lane) {
    ld = ld_;
    left = rows - r0;
    const int r = lane & 15, g = lane >> 4;
    if constexpr (KC) {
      base = (const E*)p + off0 + r0 * ld;
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const int64_t row = 16 * i + r < left ? 16 * i + r : left - 1;
        off[i] = (uint32_t)((row * ld + (ES == 4 ? 4 : 8) * g) * ES);
      }
    } else {
      // a vector may run up to NT - 1 elements past its row's end: into the
      // next row, whose values only reach results that are dropped
      base = (const E*)p + off0 + r0;
      const int64_t col = NT * r < left ? NT * r : left - 1;
      off[0] = (uint32_t)(((ES == 4 ? 4 : 8) * g * ld + col) * ES);
    }
  }
  // K-steps from the first that load() may take: whole ones, and on an edge
  // tile of an M/N-contiguous operand none of the last rows from which a
  // vector would run past the matrix's last element (the last row; several of
  // rows shorter than a vector; all where rows coincide)
  __device__ __forceinline__ int64_t whole_steps(int64_t K) const {
    if (KC || NT == 1 || left >= 16 * NT) return K / 32;
    if (ld <= 0) return 0;
    const int64_t rows = K - (ld >= NT ? 1 : (NT - 1 + ld - 1) / ld);
    return rows > 0 ? rows / 32 : 0;
  }
  // p: base + batch offset + the K-step's origin
  __device__ __forceinline__ void load(typename Op::Raw (&x)[NT], const E* p) const {
    if constexpr (KC) {
#pragma unroll
      for (int i = 0; i < NT; ++i) {
        const char* q = (const char*)p + off[i];
        if constexpr (ES == 2) {
          __builtin_memcpy(&x[i], &(const ev8&)*(const ev8*)q, 16);
        } else {
        const ev4 lo = *(const ev4*)q, hi = *(const ev4*)(q + 16 * ES);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          Op::set(x[i], e, lo[e]);
          Op::set(x[i], 4 + e, hi[e]);
        }
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const char* q = (const char*)(p + small_k<T>(0, e) * ld) + off[0];
        if constexpr (NT == 1) {
          Op::set(x[0], e, *(const E*)q);
        } else {
          const evn v = *(const evn*)q;
#pragma unroll
          for (int i = 0; i < NT; ++i) Op::set(x[i], e, v[i]);
        }
      }
    }
  }
  // any K-step, element by element: zero past K, the last row past the matrix
  __device__ __forceinline__ void load_edge(typename Op::Raw (&x)[NT], int64_t boff, int64_t k0, int64_t K, int lane) const {
    const int g = lane >> 4, r = lane & 15;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int64_t k = k0 + small_k<T>(g, e), kc = k < K ? k : K - 1;
        const int64_t row = KC ? 16 * i + r : NT * r + i, rc = row < left ? row : left - 1;
        const E v = base[boff + (KC ? rc * ld + kc : kc * ld + rc)];
        Op::set(x[i], e, k < K ? v : (E)0);
      }
  }
};

// The tile of block `bid` of `nb` by WK waves; TM x TN tiles of 16x16, DEPTH
// K-steps in flight a wave. ACT: with p.act and p.z.
template <typename T, bool A_KC, bool B_KC, int TM, int TN, int WK, int DEPTH, bool ACT>
struct SmallGemm {
  static constexpr int BM = 16 * TM, BN = 16 * TN, NTHR = 64 * WK;
  static constexpr int PITCH = BN + 4;  // floats per LDS row of a partial tile
  static constexpr int RUN = 8;  // K-steps an accumulator sums (256 terms)
  static_assert(RUN % DEPTH == 0, "runs of whole rounds of loads");
  static constexpr int LDS_FLOATS = WK * BM * PITCH + WK * BM;
  using Op = SmallOperand<T>;
  using E = typename Op::Elem;

  static __device__ __forceinline__ void run(const GemmParams& p, uint32_t bid, uint32_t nb, float* lds) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, g = lane >> 4;
    // block -> (split, batch, tile), 32-bit (fewer than 2^31 blocks): a launch
    // this short feels every 64-bit division. Consecutive logical ids sit on
    // one XCD (see xcd_remap); tiles run down the shorter side, so that
    // neighbours share the longer side's panel in its L2.
    const uint32_t per = nb >> 3, rem8 = nb & 7, xcd = bid & 7;
    uint32_t logical = xcd * per + (xcd < rem8 ? xcd : rem8) + (bid >> 3);
    const uint32_t tiles = (uint32_t)p.tiles_m * (uint32_t)p.tiles_n;
    uint32_t batch = 0, split = 0, t = logical;
    if (nb > tiles) {
      const uint32_t q = logical / tiles, kc = (uint32_t)p.keep_count;
      t = logical - q * tiles;
      split = q / kc;
      batch = q - split * kc;
    }
    uint32_t tm, tn;
    if (p.tiles_m <= p.tiles_n) {
      tn = t / (uint32_t)p.tiles_m;
      tm = t - tn * (uint32_t)p.tiles_m;
    } else {
      tm = t / (uint32_t)p.tiles_n;
      tn = t - tm * (uint32_t)p.tiles_n;
    }
    const int64_t m0 = (int64_t)tm * BM, n0 = (int64_t)tn * BN;
    int64_t a_off = 0, b_off = 0, c_off = 0;
    {
      uint32_t rem = batch;
      for (int d = p.nkeep - 1; d >= 0; --d) {
        const uint32_t n = (uint32_t)p.keep_shape[d], i = rem % n;
        rem /= n;
        a_off += i * p.keep_sa[d];
        b_off += i * p.keep_sb[d];
        c_off += i * p.keep_sc[d];
      }
    }
    const uint32_t R = (uint32_t)p.red_count;
    SmallLoader<T, A_KC, TM> la;
    SmallLoader<T, B_KC, TN> lb;
    la.init(p.a, a_off, m0, p.lda, p.M, lane);
    lb.init(p.b, b_off, n0, p.ldb, p.N, lane);
    auto red_off = [&](uint32_t r, int64_t& ra, int64_t& rb) {
      ra = rb = 0;
      for (int d = p.nred - 1; d >= 0; --d) {
        const uint32_t n = (uint32_t)p.red_shape[d], i = r % n;
        r /= n;
        ra += i * p.red_sa[d];
        rb += i * p.red_sb[d];
      }
    };
    f32x4 acc[TM][TN];
    float cs[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) cs[i] = 0.f;
    // fp32: every other wave's share is summed negated (see DmaMma<float>)
    const bool negated = Op::SPLIT && (wave & 1);
    const float b_scale = negated ? -X6_SCALE : X6_SCALE;
    const bool cs_on = !A_KC && p.colsum != nullptr && n0 == 0;
    // the wave's partial tile in LDS: stored, or added to what it has deposited
    // before (every element is one lane's alone)
    float* const part = lds + wave * BM * PITCH;
    auto deposit = [&](bool add, float unscale) {
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        float* row = part + (A_KC ? 16 * i + r16 : TM * r16 + i) * PITCH;
#pragma unroll
        for (int q = 0; q < TN; ++q) acc[i][q] *= unscale;
        if constexpr (B_KC || TN == 1) {
#pragma unroll
          for (int q = 0; q < TN; ++q) {
            f32x4* at = (f32x4*)&row[16 * q + 4 * g];
            *at = add ? *at + acc[i][q] : acc[i][q];
          }
        } else {
          // tile q's column r is column TN r + q
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            typedef float f32xTN __attribute__((ext_vector_type(TN)));
            f32xTN v;
#pragma unroll
            for (int q = 0; q < TN; ++q) v[q] = acc[i][q][e];
            f32xTN* at = (f32xTN*)&row[TN * (4 * g + e)];
            *at = add ? *at + v : v;
          }
        }
      }
    };
    auto clear = [&]() {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int q = 0; q < TN; ++q) acc[i][q] = f32x4{};
    };
    auto not_finite = [&]() {
      float z = 0.f;  // 0 x finite = 0, 0 x (inf or NaN) = NaN
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int q = 0; q < TN; ++q)
#pragma unroll
          for (int e = 0; e < 4; ++e) z = __builtin_fmaf(acc[i][q][e], 0.f, z);
      return z != z;
    };
    auto multiply = [&](auto plain, const typename Op::Raw (&xa)[TM], const typename Op::Raw (&xb)[TN]) {
      if constexpr (!A_KC) {
        // (the second pass of a share: the first has summed them)
        if (cs_on && (!decltype(plain)::value || p.plain)) {
#pragma unroll
          for (int i = 0; i < TM; ++i) cs[i] += Op::sum(xa[i]);
        }
      }
      if constexpr (decltype(plain)::value) {
#pragma unroll
        for (int i = 0; i < TM; ++i) std::conditional_t<decltype(plain)::value, Op, void>::plain(xa[i], xb, acc[i]);
      } else {
        typename Op::Frag fb[TN];
#pragma unroll
        for (int q = 0; q < TN; ++q) fb[q] = Op::frag(xb[q], b_scale);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const typename Op::Frag fa = Op::frag(xa[i], X6_SCALE);
          Op::mfma(fa, fb, acc[i]);
        }
      }
    };
    // The K-steps of every summed batch element: KF that load() takes, then
    // the rest (one or two, all of them where rows coincide) element by
    // element. This wave takes its share of the first and of the second
    // (32-bit: the host bounds their number).
    const uint32_t KS = (uint32_t)((p.K + 31) / 32);
    uint32_t KF = 0;
    if (p.K > 0) {
      const int64_t fa = la.whole_steps(p.K), fb = lb.whole_steps(p.K);
      KF = (uint32_t)(fa < fb ? fa : fb);
    }
    struct Share {
      uint32_t lo, hi;
    };
    auto share = [&](uint32_t steps, uint32_t w) -> Share {  // of this block's wave w
      uint32_t b0 = 0, n = steps;
      if (p.splits > 1) {
        b0 = (uint32_t)((uint64_t)steps * split / (uint32_t)p.splits);
        n = (uint32_t)((uint64_t)steps * (split + 1) / (uint32_t)p.splits) - b0;
      }
      return {b0 + (uint32_t)((uint64_t)n * w / WK), b0 + (uint32_t)((uint64_t)n * (w + 1) / WK)};
    };
    // The wave's share, deposited; whether a sum of it is not finite.
    auto take_share = [&](auto plain) {
      const float unscale = decltype(plain)::value ? 1.f : negated ? -Op::UNSCALE : Op::UNSCALE;
      bool bad = false, deposited = false;
      clear();
      const Share f = share(KF * R, wave);
      const int n = (int)(f.hi - f.lo);
      uint32_t cr = 0, ck = f.lo;  // the next K-step to load
      if (R > 1 && KF > 0) {
        cr = f.lo / KF;
        ck = f.lo - cr * KF;
      }
      const E *pa = la.base, *pb = lb.base;
      const int64_t da = A_KC ? 32 : 32 * p.lda, db = B_KC ? 32 : 32 * p.ldb;
      auto seek = [&]() {
        int64_t ra, rb;
        red_off(cr, ra, rb);
        pa = la.base + ra + ck * da;
        pb = lb.base + rb + ck * db;
      };
      typename Op::Raw xa[DEPTH][TM], xb[DEPTH][TN];
      int left = n;  // steps not yet loaded
      auto load_next = [&](int u) {
        if (left <= 0) return;
        --left;
        la.load(xa[u], pa);
        lb.load(xb[u], pb);
        pa += da;
        pb += db;
        if (R > 1 && ++ck == KF) {
          ck = 0;
          if (++cr < R) seek();
        }
      };
      if (n > 0) {
        seek();
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) load_next(u);
#pragma unroll 1
        for (int s = 0; s < n; s += DEPTH) {
          // a long share is summed in runs of RUN K-steps, so that an
          // accumulator takes no more roundings than those of a contraction
          // split over the grid (fp32, K = 8144 in 8 shares: 4.9e-7 off 64
          // bits, in runs 2.4e-7; 1% of the time at 16 steps a share)
          if (s > 0 && s % RUN == 0) {
            bad |= Op::SPLIT && not_finite();
            deposit(deposited, unscale);
            deposited = true;
            clear();
          }
#pragma unroll
          for (int u = 0; u < DEPTH; ++u) {
            if (u == 0 || s + u < n) multiply(plain, xa[u], xb[u]);
            load_next(u);
          }
        }
      }
      if (KF < KS) {
        const uint32_t edges = KS - KF;
        const Share e = share(edges * R, wave);
#pragma unroll 1
        for (uint32_t i = e.lo; i < e.hi; ++i) {
          const uint32_t r = i / edges, st = KF + (i - r * edges);
          int64_t ra, rb;
          red_off(r, ra, rb);
          la.load_edge(xa[0], ra, (int64_t)st * 32, p.K, lane);
          lb.load_edge(xb[0], rb, (int64_t)st * 32, p.K, lane);
          multiply(plain, xa[0], xb[0]);
        }
      }
      bad |= Op::SPLIT && not_finite();
      deposit(deposited, unscale);
      return bad;
    };
    bool bad = true;
    if (!Op::SPLIT || !p.plain) bad = take_share(std::false_type{});
    if constexpr (Op::SPLIT) {
      // what the split does not serve: the share again, by the fp32
      // instructions (16 x 4096 x 4096 forward 23.4 us, with one NaN in x
      // 24.7, all NaN 37; a thread for each result instead: 1.5 ms)
      if (__any(bad)) take_share(std::true_type{});
    }

    // ---- the waves' partial tiles meet in LDS
    float* const cs_part = lds + WK * BM * PITCH;
    if constexpr (!A_KC) {
      if (cs_on) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          float v = cs[i];
          v += __shfl_xor(v, 16);
          v += __shfl_xor(v, 32);
          if (g == 0) cs_part[wave * BM + TM * r16 + i] = v;
        }
      }
    }
    __syncthreads();
    const bool to_partial = p.splits > 1;
    if (cs_on) {
      for (int c = tid; c < BM; c += NTHR) {
        float s = 0.f;
        for (int w = 0; w < WK; ++w) s += cs_part[w * BM + c];
        const int64_t m = m0 + c;
        if (m < p.M) {
          if (to_partial) p.colsum_part[(int64_t)split * p.M + m] = s;
          else p.colsum[m] = p.accumulate ? p.colsum[m] + s : s;
        }
      }
    }
    float* const C = to_partial ? p.partial + (int64_t)split * p.partial_stride + batch * p.M * p.N : p.c + c_off;
    const int64_t ldc = to_partial ? p.N : p.ldc;
    // four consecutive columns a thread; 16-byte accesses where rows allow
    const bool vec = (p.N & 3) == 0 && (ldc & 3) == 0 && ((uintptr_t)C & 15) == 0 &&
                     (!p.z || ((p.ldz & 3) == 0 && ((uintptr_t)p.z & 15) == 0));
#pragma unroll 1
    for (int o = tid; o < BM * BN / 4; o += NTHR) {
      const int mr = o / (BN / 4), nr = o % (BN / 4) * 4;
      const int64_t m = m0 + mr, n = n0 + nr;
      if (m >= p.M || n >= p.N) continue;
      f32x4 v = *(const f32x4*)&lds[mr * PITCH + nr];
#pragma unroll
      for (int w = 1; w < WK; ++w) v += *(const f32x4*)&lds[(w * BM + mr) * PITCH + nr];
      float* c = C + m * ldc + n;
      float* z = p.z ? p.z + m * p.ldz + n : nullptr;
      const int cnt = p.N - n < 4 ? (int)(p.N - n) : 4;
      if (!to_partial) {
        if (p.bias)
          for (int e = 0; e < cnt; ++e) v[e] += p.bias[n + e];
        if constexpr (ACT) {
          if (z) {
            if (vec) *(f32x4*)z = v;
            else
              for (int e = 0; e < cnt; ++e) z[e] = v[e];
          }
        }
        if constexpr (ACT)
          for (int e = 0; e < 4; ++e) v[e] = act_apply(p.act, v[e]);
        if (p.accumulate)
          for (int e = 0; e < cnt; ++e) v[e] += c[e];
      }
      if (vec) *(f32x4*)c = v;
      else
        for (int e = 0; e < cnt; ++e) c[e] = v[e];
    }
  }
};

template <typename T, bool A_KC, bool B_KC, int TM, int TN, int WK, int DEPTH, bool ACT>
__global__ __launch_bounds__(64 * WK) __attribute__((amdgpu_waves_per_eu(WK / 4, WK / 4)))
void gemm_small_kernel(const GemmParams p) {
  using G = SmallGemm<T, A_KC, B_KC, TM, TN, WK, DEPTH, ACT>;
  __shared__ __attribute__((aligned(16))) float lds[G::LDS_FLOATS];
  G::run(p, blockIdx.x, gridDim.x, lds);
}

// dX = dY W and dW = dY^T X (with db) of a small layer in one launch: blocks
// 0 .. nb_dx-1 take dX's tiles, the others dW's.
template <typename T, int TM, int TN, int WK, int DEPTH>
__global__ __launch_bounds__(64 * WK) __attribute__((amdgpu_waves_per_eu(WK / 4, WK / 4)))
void gemm_small_bwd_kernel(const GemmParams pdx, const GemmParams pdw, uint32_t nb_dx) {
  using X = SmallGemm<T, true, false, TM, TN, WK, DEPTH, false>;
  using W = SmallGemm<T, false, false, TM, TN, WK, DEPTH, false>;
  __shared__ __attribute__((aligned(16))) float lds[X::LDS_FLOATS > W::LDS_FLOATS ? X::LDS_FLOATS : W::LDS_FLOATS];
  if (blockIdx.x < nb_dx) X::run(pdx, blockIdx.x, nb_dx, lds);
  else W::run(pdw, blockIdx.x - nb_dx, gridDim.x - nb_dx, lds);
}

// Launches, for one element type. Tiles: 64x64 and 32x32 by 8 waves, 16x16 by 16.
template <typename T>
struct SmallLaunch {
  static bool prepare(const GemmParams& p, int tile, GemmParams* q, int64_t* blocks) {
    *q = p;
    q->tiles_m = (int32_t)((p.M + tile - 1) / tile);
    q->tiles_n = (int32_t)((p.N + tile - 1) / tile);
    *blocks = (int64_t)q->tiles_m * q->tiles_n * p.keep_count * p.splits;
    return *blocks <= 0x7fffffff;
  }
  template <bool A_KC, bool B_KC, bool ACT = false>
  static hipError_t layout(const GemmParams& p, int tile, hipStream_t stream) {
    GemmParams q;
    int64_t blocks;
    if (!prepare(p, tile, &q, &blocks)) return hipErrorInvalidConfiguration;
    if (blocks <= 0) return hipSuccess;
    if (tile == 64)
      hipLaunchKernelGGL((gemm_small_kernel<T, A_KC, B_KC, 4, 4, 8, 1, ACT>), dim3((unsigned)blocks), dim3(512), 0, stream, q);
    else if (tile == 32)
      hipLaunchKernelGGL((gemm_small_kernel<T, A_KC, B_KC, 2, 2, 8, 4, ACT>), dim3((unsigned)blocks), dim3(512), 0, stream, q);
    else
      hipLaunchKernelGGL((gemm_small_kernel<T, A_KC, B_KC, 1, 1, 16, 4, ACT>), dim3((unsigned)blocks), dim3(1024), 0, stream, q);
    return hipGetLastError();
  }
  static hipError_t run(const GemmParams& p, bool a_kc, bool b_kc, int tile, hipStream_t stream) {
    if (p.act || p.z) return layout<true, true, true>(p, tile, stream);  // (NT only)
    if (a_kc) return b_kc ? layout<true, true>(p, tile, stream) : layout<true, false>(p, tile, stream);
    return b_kc ? layout<false, true>(p, tile, stream) : layout<false, false>(p, tile, stream);
  }
  static hipError_t bwd(const GemmParams& pdx, const GemmParams& pdw, int tile, hipStream_t stream) {
    GemmParams x, w;
    int64_t bx, bw;
    if (!prepare(pdx, tile, &x, &bx) || !prepare(pdw, tile, &w, &bw) || bx + bw > 0x7fffffff)
      return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)(bx + bw));
    if (bx + bw <= 0) return hipSuccess;
    if (tile == 64)
      hipLaunchKernelGGL((gemm_small_bwd_kernel<T, 4, 4, 8, 1>), grid, dim3(512), 0, stream, x, w, (uint32_t)bx);
    else if (tile == 32)
      hipLaunchKernelGGL((gemm_small_bwd_kernel<T, 2, 2, 8, 4>), grid, dim3(512), 0, stream, x, w, (uint32_t)bx);
    else
      hipLaunchKernelGGL((gemm_small_bwd_kernel<T, 1, 1, 16, 4>), grid, dim3(1024), 0, stream, x, w, (uint32_t)bx);
    return hipGetLastError();
  }
};

}  // namespace gemm
}  // namespace mt
