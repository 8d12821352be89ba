// Many-row GEMM with 256-column blocks whose weight operand never passes
// through LDS.
//
// What bounds it: in the 128 x 128 ring kernels a wave reads both operands of
// its 64 x 32 tile from LDS, 96 KiB per CU and k-block against 512 cycles of
// MFMA, so the LDS port sets their rate (about 65 % of the matrix cores').
// The weights are stored in operand order, so here each of the four waves
// loads the fragments of its own 64 columns straight into registers (no other
// wave of the block needs them, and fp8 codes are expanded once), and only
// the 16 MT x 64 activation tile is staged in LDS, which all four waves read:
// at MT = 8 that is 64 KiB of LDS reads per 1024 cycles of MFMA.
//
// Both operands of k-block kb + NS - 1 are requested while kb is computed.
// NS = 2 keeps a wave within 256 registers, so that two blocks share a CU and
// cover each other's waits; NS = 4 is for grids of at most one block per CU,
// where weights come cold and nothing else hides their latency.  Counters: the
// long grids keep the matrix cores 42 to 47 % busy (gate/up 816 x 2048 x 32768
// bf16 1,194 TFLOP/s, 3264 x 1024 x 8192 fp8 1,132), LDS 11 to 12 % (the ring
// 29 % at 720 TFLOP/s), the vector ALU 5 to 8 %, and take in 13 bytes of bf16
// weights per CU and cycle; the one-block grids 11 to 26 %, 3 to 7 %, 2 to 4 %
// and 10 to 16 bytes.  So no unit is saturated: what is left is the wait
// for each k-block's loads, with one or two waves per SIMD to cover it.  Deeper
// rings (6, 8 stages), K halved over two wave groups, loads spread between the
// MFMAs and a contiguous weight order all measured the same or slower.
//
// The MFMAs run with the weights as the first operand: accumulator v of lane
// l is column 16 t + 4 (l / 16) + v of row 16 m + l % 16, so a lane's four
// values are consecutive columns and every epilogue access is 8 or 16 bytes.
#pragma once

#include "gemm_tile.hpp"

#include <type_traits>

namespace phyai {
namespace {

// Two groups of four bf16 columns, x and y, each spread over the four lane
// groups of a row: afterwards even lane groups hold eight consecutive columns
// of x and odd ones of y (columns 8 (lg / 2) .. of half lg % 2), so that a row
// leaves in 16-byte stores, 64 contiguous bytes per instruction.
__device__ __forceinline__ uint4 join_halves(const float (&x)[4], const float (&y)[4]) {
  const auto a = __builtin_amdgcn_permlane16_swap(pack_bf16x2(x[0], x[1]), pack_bf16x2(y[0], y[1]), false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(pack_bf16x2(x[2], x[3]), pack_bf16x2(y[2], y[3]), false, false);
  return make_uint4(a[0], b[0], a[1], b[1]);
}

// Epilogues of a wave's (16 MT) x 64 tile: row0 the tile's first row, p0 the
// first of its two pair tiles, lr = lane % 16 the row within each 16, lg =
// lane / 16 the group of four columns, acc[m][t] as above (t: the 16-column
// halves of the two pair tiles in order), already scaled.
template <int ACT, typename OutT, int MT>
__device__ __forceinline__ void wide_store(const GemmArgs& g, const EpiStore<OutT>& e, f32x4 (&acc)[MT][4], int row0,
                                              int p0, int lr, int lg) {
  f32x4 b[4], rv[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int col = 32 * p0 + 16 * t + 4 * lg;
    b[t] = e.bias ? *reinterpret_cast<const f32x4*>(e.bias + col) : f32x4{0.f, 0.f, 0.f, 0.f};
    rv[t] = e.rowvec ? *reinterpret_cast<const f32x4*>(e.rowvec + col) : f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int row = row0 + 16 * m + lr;
    if (row >= g.R) continue;
    const int orow = e.grp > 0 ? (row / e.grp) * e.grp_stride + e.grp_off + row % e.grp : row;
    OutT* o = e.out + (int64_t)orow * e.ldo + 32 * p0;
#pragma unroll
    for (int pp = 0; pp < 2; ++pp) {
      float v[2][4];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          v[t][i] = apply_act<OutT>(ACT, acc[m][2 * pp + t][i] + b[2 * pp + t][i] + rv[2 * pp + t][i]);
      if constexpr (std::is_same<OutT, float>::value) {
        ActIO<OutT>::store4(o + 32 * pp + 4 * lg, v[0]);
        ActIO<OutT>::store4(o + 32 * pp + 16 + 4 * lg, v[1]);
      } else {
        *reinterpret_cast<uint4*>(o + 32 * pp + 16 * (lg % 2) + 8 * (lg / 2)) = join_halves(v[0], v[1]);
      }
    }
  }
}

// The activation is chosen once per wave: tested per value it doubled the
// epilogue (64 x 256 GELU tile 9.3 -> 4.8 kcycles).
template <typename OutT, int MT>
__device__ __forceinline__ void wide_epilogue(const GemmArgs& g, const EpiStore<OutT>& e, f32x4 (&acc)[MT][4], int row0,
                                              int p0, int lr, int lg, bf16_t*) {
  if (e.act == ACT_GELU) wide_store<ACT_GELU>(g, e, acc, row0, p0, lr, lg);
  else if (e.act == ACT_SWISH) wide_store<ACT_SWISH>(g, e, acc, row0, p0, lr, lg);
  else wide_store<ACT_NONE>(g, e, acc, row0, p0, lr, lg);
}

template <int MT>
__device__ __forceinline__ void wide_epilogue(const GemmArgs& g, const EpiResid& e, f32x4 (&acc)[MT][4], int row0,
                                              int p0, int lr, int lg, bf16_t*) {
  f32x4 b[4], gt[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int col = 32 * p0 + 16 * t + 4 * lg;
    b[t] = e.bias ? *reinterpret_cast<const f32x4*>(e.bias + col) : f32x4{0.f, 0.f, 0.f, 0.f};
    gt[t] = e.gate ? *reinterpret_cast<const f32x4*>(e.gate + col) : f32x4{1.f, 1.f, 1.f, 1.f};
  }
  // the residual rows of two 16-row groups are requested before their stores
  // (rows past R read row R - 1)
#pragma unroll
  for (int m0 = 0; m0 < MT; m0 += 2) {
    f32x4 hv[2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      if (m0 + m >= MT) continue;
      const float* h = e.h + (int64_t)min(row0 + 16 * (m0 + m) + lr, g.R - 1) * e.ldh + 32 * p0 + 4 * lg;
#pragma unroll
      for (int t = 0; t < 4; ++t) hv[m][t] = *reinterpret_cast<const f32x4*>(h + 16 * t);
    }
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const int row = row0 + 16 * (m0 + m) + lr;
      if (m0 + m >= MT || row >= g.R) continue;
      float* h = e.h + (int64_t)row * e.ldh + 32 * p0 + 4 * lg;
#pragma unroll
      for (int t = 0; t < 4; ++t)
        *reinterpret_cast<f32x4*>(h + 16 * t) = hv[m][t] + (acc[m0 + m][t] + b[t]) * gt[t];
    }
  }
}

template <bool LO, int MT>
__device__ __forceinline__ void wide_geglu(const GemmArgs& g, const EpiGeglu<bf16_t>& e, f32x4 (&acc)[MT][4], int row0,
                                           int p0, int lr, int lg) {
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int row = row0 + 16 * m + lr;
    if (row >= g.R) continue;
    float v[2][4], lo[2][4];
#pragma unroll
    for (int pp = 0; pp < 2; ++pp)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float z = acc[m][2 * pp][i];
        v[pp][i] = (LO ? gelu_tanh_f(z) : gelu_tanh_bf16(z)) * acc[m][2 * pp + 1][i];
        if constexpr (LO) lo[pp][i] = v[pp][i] - ActIO<bf16_t>::round(v[pp][i]);
      }
    const int64_t o = (int64_t)row * e.ldo + 16 * (p0 + lg % 2) + 8 * (lg / 2);
    *reinterpret_cast<uint4*>(e.out + o) = join_halves(v[0], v[1]);
    if constexpr (LO) *reinterpret_cast<uint4*>(e.lo + o) = join_halves(lo[0], lo[1]);
  }
}
template <int MT>
__device__ __forceinline__ void wide_epilogue(const GemmArgs& g, const EpiGeglu<bf16_t>& e, f32x4 (&acc)[MT][4],
                                              int row0, int p0, int lr, int lg, bf16_t*) {
  wide_geglu<false>(g, e, acc, row0, p0, lr, lg);
}
template <int MT>
__device__ __forceinline__ void wide_epilogue(const GemmArgs& g, const EpiGegluLo& e, f32x4 (&acc)[MT][4], int row0,
                                              int p0, int lr, int lg, bf16_t*) {
  wide_geglu<true>(g, e, acc, row0, p0, lr, lg);
}

// A wave's 64 columns lie in one head, so whether they are Q, K or V is known
// once per tile.  V goes through LDS (`st`, kVStage elements per wave), 64 rows
// at a time, so that each store writes 64 consecutive keys of one V^T row.
template <int MT>
__device__ __forceinline__ void wide_epilogue(const GemmArgs& g, const EpiQkv<bf16_t>& e, f32x4 (&acc)[MT][4], int row0,
                                              int p0, int lr, int lg, bf16_t* st) {
  const int D = e.D, tiles = D / 32, head = p0 / tiles;
  const int i0 = 16 * (p0 % tiles) + 4 * lg;      // first of the lane's dims in pair tile p0 (p0 + 1: + 16)
  if (e.bias) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const f32x4 b = *reinterpret_cast<const f32x4*>(e.bias + head * D + i0 + 16 * (t / 2) + (t % 2) * (D / 2));
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m][t] += b;
    }
  }
  if (head >= e.nq + e.nkv) {
    const int lane = 16 * lg + lr;
#pragma unroll
    for (int m0 = 0; m0 < MT; m0 += 4) {
#pragma unroll
      for (int m = m0; m < (m0 + 4 < MT ? m0 + 4 : MT); ++m)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            st[(16 * t + 4 * lg + i) * EpiQkv<bf16_t>::kVRow + 16 * (m - m0) + lr] = f32_to_bf16(acc[m][t][i]);
      __builtin_amdgcn_s_waitcnt(0xC07F);         // the wave's LDS writes are done (lgkmcnt 0)
      const int row = row0 + 16 * m0 + lane;
      if (lane < 16 * (MT - m0) && row < g.R) {
        const int key = (e.keys_after_prefix ? e.desc->prefix_len[row / e.M] : 0) + row % e.M;
        bf16_t* vrow = e.vt + ((int64_t)(row / e.M) * e.nkv + (head - e.nq - e.nkv)) * D * e.ldk + key;
#pragma unroll 8
        for (int col = 0; col < 64; ++col) {
          const int d = 16 * (p0 % tiles + col / 32) + col % 16 + ((col / 16) % 2) * (D / 2);
          vrow[(int64_t)d * e.ldk] = st[col * EpiQkv<bf16_t>::kVRow + lane];
        }
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);         // ... and read back before the next 64 rows
    }
    return;
  }
  const bool rot = e.rope != 0;
  const bool isq = head < e.nq;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int row = row0 + 16 * m + lr;
    if (row >= g.R) continue;
    bf16_t* dst;
    if (isq) {
      dst = e.q + (int64_t)row * e.nq * D + head * D;
    } else {
      const int key = (e.keys_after_prefix ? e.desc->prefix_len[row / e.M] : 0) + row % e.M;
      dst = e.kall + (((int64_t)(row / e.M) * e.nkv + (head - e.nq)) * e.ldk + key) * D;
    }
    f32x4 cs[2][2];                               // (cos, sin) of the lane's 4 dims, two pair tiles
    if (rot) {
#pragma unroll
      for (int pp = 0; pp < 2; ++pp)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          cs[pp][j] = *reinterpret_cast<const f32x4*>(e.rope_cs + (int64_t)row * (D / 2) + i0 + 16 * pp + 2 * j);
    }
    float x1[2][4], x2[2][4];
#pragma unroll
    for (int pp = 0; pp < 2; ++pp)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float u = acc[m][2 * pp][i], w = acc[m][2 * pp + 1][i];
        x1[pp][i] = u;
        x2[pp][i] = w;
        if (rot) {
          const float c = cs[pp][i / 2][2 * (i % 2)], s = cs[pp][i / 2][2 * (i % 2) + 1];
          x1[pp][i] = u * c - w * s;
          x2[pp][i] = w * c + u * s;
        }
      }
    const int i = 16 * (p0 % tiles + lg % 2) + 8 * (lg / 2);
    *reinterpret_cast<uint4*>(dst + i) = join_halves(x1[0], x1[1]);
    *reinterpret_cast<uint4*>(dst + i + D / 2) = join_halves(x2[0], x2[1]);
  }
}

// Rows a request does not have (past its prefix length) leave as zeros.
template <int MT>
__device__ __forceinline__ void wide_epilogue(const GemmArgs& g, const EpiKV<bf16_t>& e, f32x4 (&acc)[MT][4], int row0,
                                              int p0, int lr, int lg, bf16_t*) {
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int row = row0 + 16 * m + lr;
    if (row >= g.R) continue;
    const int b = row / e.P, key = row % e.P;
    const bool ok = g.rows_per_req <= 0 || row % g.rows_per_req < g.desc->prefix_len[row / g.rows_per_req];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int col = 32 * p0 + 16 * t + 4 * lg;
      const int kv = col / (e.nkv * e.D), rem = col % (e.nkv * e.D);
      const int h = rem / e.D, i = rem % e.D;
      float v[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = ok ? acc[m][t][j] : 0.f;
      const int64_t lo = (kv / 2) * e.layer_stride;
      if (kv % 2 == 0) {
        ActIO<bf16_t>::store4(e.kall + lo + (((int64_t)b * e.nkv + h) * e.ldk + key) * e.D + i, v);
      } else {
        bf16_t* dst = e.vt + lo + (((int64_t)b * e.nkv + h) * e.D + i) * e.ldk + key;
#pragma unroll
        for (int j = 0; j < 4; ++j) dst[(int64_t)j * e.ldk] = f32_to_bf16(v[j]);
      }
    }
  }
}

template <class Epi> struct IsQkv : std::false_type {};
template <typename T> struct IsQkv<EpiQkv<T>> : std::true_type {};

// Tiles of 16 MT rows x 256 columns in bands of four column tiles, row by row
// within a band; XCD x takes the x-th eighth of that order, so that its L2
// serves one band's weights to all of its blocks (3264 x 1024 x 8192: 68 us
// against 88 with all column tiles in one band).
constexpr int kWideBand = 4;

template <class Epi, int WK, int MT, int NS, bool TWO>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NS == 2 ? 2 : 1))) void
gemm_wide_kernel(GemmArgs g, Epi epi) {
  constexpr bool FP8 = WK == W_FP8;
  constexpr int FB = FP8 ? 1024 : 2048;       // bytes per (pair, half) fragment per k-block
  constexpr int BW = FP8 ? 1 : 2;             // 16-byte loads per fragment and lane
  constexpr int ABLK = 2 * MT;                // 1 KiB blocks of an activation tile
  constexpr int LA1 = (ABLK + 3) / 4;         // copies per wave and operand term (a last one may repeat a block)
  constexpr int TERMS = TWO ? 2 : 1;
  constexpr int LOADS = LA1 * TERMS + 4 * BW; // per wave and k-block
  constexpr int STAGE = ABLK * 1024 * TERMS;
  constexpr int VBYTES = IsQkv<Epi>::value ? 4 * EpiQkv<bf16_t>::kVStage * 2 : 0;
  __shared__ __attribute__((aligned(1024))) uint8_t ring[NS * STAGE > VBYTES ? NS * STAGE : VBYTES];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int wv = __builtin_amdgcn_readfirstlane(wave);
  const int lr = lane % 16, lg = lane / 16;
  const int mtiles = (g.R + 16 * MT - 1) / (16 * MT), ntiles = g.NPT / 8;
  const int T = mtiles * ntiles, per = (T + 7) / 8;
  const int k8 = blockIdx.x / 8, t = (blockIdx.x % 8) * per + k8;
  if (k8 >= per || t >= T) return;
  const int bi = t / (mtiles * kWideBand), rem = t - bi * mtiles * kWideBand;
  const int bw = min(kWideBand, ntiles - bi * kWideBand);
  const int m0 = rem / bw * 16 * MT, pt0 = (bi * kWideBand + rem % bw) * 8 + 2 * wv;
  // K slice blockIdx.y of gridDim.y (split K: raw sums to split_out)
  const int nkt = g.K / 64;
  const int kb0 = (int)((int64_t)nkt * blockIdx.y / gridDim.y);
  const int nkb = (int)((int64_t)nkt * (blockIdx.y + 1) / gridDim.y) - kb0;

  // bases are wave-uniform (scalar registers), lanes add 32-bit byte offsets
  const uint8_t* abase[TERMS];
  uint32_t aoff[LA1];
  {
    const bf16_t* A = g.A_ind ? static_cast<const bf16_t*>(*g.A_ind) + g.a_off : static_cast<const bf16_t*>(g.A);
    const int64_t base = (int64_t)m0 * g.lda + kb0 * 64;
    abase[0] = reinterpret_cast<const uint8_t*>(A + base);
    if (TWO) abase[TERMS - 1] = reinterpret_cast<const uint8_t*>(static_cast<const bf16_t*>(g.A_lo) + base);
#pragma unroll
    for (int i = 0; i < LA1; ++i) {
      const int row = 8 * min(4 * i + wv, ABLK - 1) + lane / 8;
      aoff[i] = 2 * (uint32_t)((min(m0 + row, g.R - 1) - m0) * g.lda + 8 * ((lane % 8) ^ aswz(row)));
    }
  }
  const uint8_t* bbase = static_cast<const uint8_t*>(g.W) + ((int64_t)pt0 * nkt + kb0) * 2 * FB;
  const uint32_t boff = lane * (16 * BW);

  static_assert(NS == 2 || NS == 4, "two or four stages");
  u32x4_t b[NS == 2 ? 1 : NS][4][BW];
  auto issue = [&](uint8_t* base, u32x4_t (&bs)[4][BW], int kb) {
#pragma unroll
    for (int q = 0; q < TERMS; ++q)
#pragma unroll
      for (int i = 0; i < LA1; ++i)
        dma16_off(abase[q] + (int64_t)kb * 128, aoff[i],
                  (lds_void_t*)(base + q * ABLK * 1024 + min(4 * i + wv, ABLK - 1) * 1024));
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
      for (int w = 0; w < BW; ++w)
        bs[n][w] = gload16_off(bbase + ((int64_t)(n / 2) * nkt + kb) * (2 * FB) + (n % 2) * FB + 16 * w, boff);
    __builtin_amdgcn_sched_barrier(0);
  };

  f32x4 acc[MT][4];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int n = 0; n < 4; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto compute = [&](const uint8_t* base, const u32x4_t (&bs)[4][BW]) {
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      bf16x8 bf[4];
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        if constexpr (FP8) bf[n] = st == 0 ? fp8x8_to_bf16x8(bs[n][0].x, bs[n][0].y)
                                           : fp8x8_to_bf16x8(bs[n][0].z, bs[n][0].w);
        else bf[n] = __builtin_bit_cast(bf16x8, bs[n][BW == 2 ? st : 0]);
      }
#pragma unroll
      for (int q = 0; q < TERMS; ++q) {
        const bf16_t* As = reinterpret_cast<const bf16_t*>(base + q * ABLK * 1024);
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const int row = 16 * m + lr;
          const bf16x8 af = *reinterpret_cast<const bf16x8*>(As + row * 64 + 8 * ((4 * st + lg) ^ aswz(row)));
#pragma unroll
          for (int n = 0; n < 4; ++n) acc[m][n] = mfma16x16x32(bf[n], af, acc[m][n]);
        }
      }
    }
    // each activation fragment is read three MFMA groups (192 cycles) ahead of
    // its use; left to itself the compiler reads them all first and spills
    constexpr int NF = 2 * MT * TERMS, AHEAD = 3;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // DS read
#pragma unroll
    for (int i = 0; i < NF; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);                                   // MFMA
      if (i < NF - AHEAD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  if constexpr (NS == 2) {
    issue(ring, b[0], 0);
    for (int kb = 0; kb < nkb; ++kb) {
      GEMM_WAIT_VMCNT(0);                     // this wave's loads of k-block kb have landed
      bare_barrier();                         // ... everyone's, and k-block kb - 1 is consumed
      u32x4_t cur[4][BW];
#pragma unroll
      for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int w = 0; w < BW; ++w) cur[n][w] = b[0][n][w];
      if (kb + 1 < nkb) issue(ring + ((kb + 1) & 1) * STAGE, b[0], kb + 1);
      compute(ring + (kb & 1) * STAGE, cur);
    }
  } else {
    // Four stages, at least three k-blocks (the launch rule).  Whether a step
    // requests another k-block is known where it stands: behind a test the
    // compiler could not count the loads in flight, and its waits for the
    // weight registers would take in the next k-blocks too (3264 x 4096 x 1024:
    // 28 -> 40 us).  FLY: later k-blocks that may still be in flight.
    auto step = [&](auto slot, auto fly, auto more, int kb) {
      constexpr int S = decltype(slot)::value;
      GEMM_WAIT_VMCNT(decltype(fly)::value * LOADS);
      bare_barrier();
      if constexpr (decltype(more)::value) issue(ring + (S + 3) % 4 * STAGE, b[(S + 3) % NS], kb + 3);
      compute(ring + S * STAGE, b[S % NS]);
    };
    constexpr std::integral_constant<int, 0> c0;
    constexpr std::integral_constant<int, 1> c1;
    constexpr std::integral_constant<int, 2> c2;
    constexpr std::integral_constant<int, 3> c3;
    constexpr std::true_type yes;
    constexpr std::false_type no;
    issue(ring, b[0], 0);
    issue(ring + STAGE, b[1], 1);
    issue(ring + 2 * STAGE, b[2 % NS], 2);
    int kb = 0;
    for (; kb + 6 < nkb; kb += 4) {
      step(c0, c2, yes, kb);
      step(c1, c2, yes, kb + 1);
      step(c2, c2, yes, kb + 2);
      step(c3, c2, yes, kb + 3);
    }
    // three to six left, three of them requested
    if (kb + 3 < nkb) {
      step(c0, c2, yes, kb);
      if (kb + 4 < nkb) {
        step(c1, c2, yes, kb + 1);
        if (kb + 5 < nkb) {
          step(c2, c2, yes, kb + 2);
          step(c3, c2, no, kb + 3);
          step(c0, c1, no, kb + 4);
          step(c1, c0, no, kb + 5);
        } else {
          step(c2, c2, no, kb + 2);
          step(c3, c1, no, kb + 3);
          step(c0, c0, no, kb + 4);
        }
      } else {
        step(c1, c2, no, kb + 1);
        step(c2, c1, no, kb + 2);
        step(c3, c0, no, kb + 3);
      }
    } else {
      step(c0, c2, no, kb);
      step(c1, c1, no, kb + 1);
      step(c2, c0, no, kb + 2);
    }
  }

  if constexpr (FP8) {
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const f32x4 sc = *reinterpret_cast<const f32x4*>(g.scale + 32 * pt0 + 16 * n + 4 * lg);
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[m][n] *= sc;
    }
  }
  if (g.split_out) {
    float* sp = g.split_out + (int64_t)blockIdx.y * g.split_stride + 32 * pt0 + 4 * lg;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      const int row = m0 + 16 * m + lr;
      if (row >= g.R) continue;
#pragma unroll
      for (int n = 0; n < 4; ++n) *reinterpret_cast<f32x4*>(sp + (int64_t)row * (32 * g.NPT) + 16 * n) = acc[m][n];
    }
    return;
  }
  if constexpr (IsQkv<Epi>::value) bare_barrier();   // the ring is free for the V staging
  wide_epilogue(g, epi, acc, m0, pt0, lr, lg,
                reinterpret_cast<bf16_t*>(ring) + (IsQkv<Epi>::value ? wave * EpiQkv<bf16_t>::kVStage : 0));
}

template <class Epi, bool TWO, int WK>
void wide_launch(const GemmArgs& g, const Epi& epi, WideTile t, hipStream_t s) {
  auto go = [&](auto mt, auto ns) {
    constexpr int MT = decltype(mt)::value, NS = decltype(ns)::value;
    const int tiles = (g.R + 16 * MT - 1) / (16 * MT) * (g.NPT / 8);
    const dim3 grid(8 * ((tiles + 7) / 8), g.split_out ? g.split_k : 1);
    hipLaunchKernelGGL((gemm_wide_kernel<Epi, WK, MT, NS, TWO>), grid, dim3(256), 0, s, g, epi);
  };
  typedef std::integral_constant<int, 2> two;
  typedef std::integral_constant<int, 4> four;
  if (t.ns == 4) {
    if (t.mt == 2) go(std::integral_constant<int, 2>{}, four{});
    else if (t.mt == 3) go(std::integral_constant<int, 3>{}, four{});
    else go(std::integral_constant<int, 4>{}, four{});
  } else {
    if (t.mt == 4) go(std::integral_constant<int, 4>{}, two{});
    else if (t.mt == 7) go(std::integral_constant<int, 7>{}, two{});
    else if (t.mt == 8) go(std::integral_constant<int, 8>{}, two{});
    else go(std::integral_constant<int, 9>{}, two{});
  }
}

}  // namespace
}  // namespace phyai
