// The whole GMaS step of narrow layers in one kernel (Section 2.2, Step 2): all K^3
// weight matrices stay in LDS, a wave takes 16 consecutive sorted outputs at a time,
// keeps their float32 sums in registers and adds every offset's products to them.
// The per-pair partial rows of the Gather -> GEMM -> Scatter form are never written or
// read, and no barrier follows the staging.
//
// Sorted neighbours mostly have the same neighbours: of the 27 offsets, a block of 16
// consecutive outputs has pairs at few (LiDAR 120k voxels: 6.2, with 2.6 pairs per
// output; the 300k-voxel room: 11.3, 3.4 pairs).  So each block is multiplied only at
// its own offsets, with zeros in the rows that have no pair there.
//
// What bounds it: the latency of a block's chain (table entries -> pairs' input rows ->
// input rows -> products -> store) over the 16 waves a CU holds beside the weights; the
// chain's first links are requested one and two blocks ahead.  Layer times against the
// separate GEMM and scatter (one launch instead of two): K = 5, 8 -> 32 channels, 60k
// voxels 38.6 -> 18.6 us; K = 3, 32 -> 32, 242k voxels 33.8 -> 23.7 us (its table, rows
// and outputs are 60 MB: 2.5 TB/s); K = 2 stride 2, 32 -> 64, 199k voxels 22.4 -> 13.6
// us, transposed 64 -> 32 18.9 -> 14.6 us, 96 -> 96 36.2 -> 21.4 us.
//
// Tried and slower, as far as the trials were kept: float32 sums in LDS (ds_add_f32, or
// read, add and write by one wave), and wider layers with their weights streamed through
// LDS, offset by offset with a barrier each, or a few offsets at a time with two row
// blocks per wave (about even with the separate steps at 64 and 128 channels, behind them
// at 256).
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace spc {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// One 16-byte operand fragment per lane: 8 16-bit or 4 float32 consecutive
// channels of row (or column) lane % 16.  KS channels per fragment and wave.
template <typename T>
struct Frag;
template <>
struct Frag<__half> {
  static constexpr int KS = 32;
  __device__ static f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <>
struct Frag<__hip_bfloat16> {
  static constexpr int KS = 32;
  __device__ static f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
// float32: four products of 4 channels each; product j takes channel j of every
// lane's four (the same for both operands, so the sum covers all 16 channels)
template <>
struct Frag<float> {
  static constexpr int KS = 16;
  __device__ static f32x4 mma(u32x4 a, u32x4 b, f32x4 c) {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[j], y[j], c, 0, 0, 0);
    return c;
  }
};

// Output vectors: 16 bytes of T from consecutive float32 sums.
template <typename T>
struct Out;
template <>
struct Out<__half> {
  static constexpr int N = 8;
  __device__ static void add(float* v, u32x4 r) {
    const f16x8 h = __builtin_bit_cast(f16x8, r);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] += (float)h[i];
  }
  __device__ static uint4 pack(const float* v) {
    f16x8 h;
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = (_Float16)v[i];
    return __builtin_bit_cast(uint4, h);
  }
};
template <>
struct Out<__hip_bfloat16> {
  static constexpr int N = 8;
  __device__ static void add(float* v, u32x4 r) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] += __uint_as_float(r[i] << 16);
      v[2 * i + 1] += __uint_as_float(r[i] & 0xFFFF0000u);
    }
  }
  __device__ static uint4 pack(const float* v) {
    __hip_bfloat16 h[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) h[i] = __float2bfloat16(v[i]);
    return *reinterpret_cast<const uint4*>(h);
  }
};
template <>
struct Out<float> {
  static constexpr int N = 4;
  __device__ static void add(float* v, u32x4 r) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] += __uint_as_float(r[i]);
  }
  __device__ static uint4 pack(const float* v) {
    return make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
  }
};



// Whether a weight is not finite: its magnitude bits reach the all-ones exponent's.
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
template <typename T>
struct Finite {
  static constexpr uint32_t kAbs = sizeof(T) == 4 ? 0x7FFFFFFFu : 0x7FFF7FFFu;
  __device__ static bool exceeded(u32x4 top) {
    bool bad = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (sizeof(T) == 4) {
        bad |= top[i] >= 0x7F800000u;
      } else {
        constexpr uint32_t inf = std::is_same<T, __half>::value ? 0x7C00u : 0x7F80u;
        bad |= (top[i] & 0xFFFFu) >= inf || (top[i] >> 16) >= inf;
      }
    }
    return bad;
  }
};

constexpr int kConvThreads = 1024;
constexpr int kConvWaves = kConvThreads / kWave;

struct ConvArgs {
  const void* x;
  const void* w;
  const int32_t* pin;     // input row of each pair
  const int32_t* omt;     // pair of (offset, sorted output), or -1
  int64_t stride;
  const uint32_t* perm;   // caller row of each sorted output (NULL: identity)
  void* y;
  const void* residual;
  int K3, n_out, c_in, c_out, relu;
  uint32_t row_bytes, x_bytes;
};

// Byte offset of rows that are not there: past the end of any input (at most 3.5 GiB),
// so that the buffer load returns zeros without a memory access.
constexpr uint32_t kNoRow = 0xF0000000u;
constexpr int64_t kMaxInputBytes = (int64_t)0xE0000000;

// MFMA column n of column tile t of NT tiles -> output channel.  16-bit types: the
// columns of two neighbouring tiles are exchanged so that a lane's sums (columns
// 4 sub .. 4 sub + 3 of each tile) are 8 consecutive channels.
template <typename T>
__host__ __device__ constexpr int conv_channel(int nt, int t, int n) {
  return (sizeof(T) == 2 && t < (nt & ~1)) ? 32 * (t >> 1) + 8 * (n >> 2) + 4 * (t & 1) + (n & 3) : 16 * t + n;
}

constexpr size_t conv_lds(int K3, int nt, int kpo, int g, int mg) {
  return (size_t)((K3 + g - 1) / g) * kpo * nt * 1024 + (size_t)kConvWaves * 64 * mg * 4;
}

// NT column tiles (the whole row).  KPO k-steps per offset, or G = 2 or 4 offsets per
// k-step where an offset's channels fill half or a quarter of one (KPO = 1): a step is
// one offset, or G of them.  MG table entries per lane: 4 MG offsets at a time.
template <typename T, int NT, int KPO, int G, int MG>
__global__ __launch_bounds__(kConvThreads) void k_conv_small(ConvArgs g) {
  using M = Frag<T>;
  constexpr int E = 16 / (int)sizeof(T);  // channels per 16-byte piece
  constexpr int SPO = 4 / G;              // 16-byte pieces of an offset per k-step
  constexpr int kOffsetGroup = 4 * MG;    // offsets at a time
  // steps whose input rows are requested together
  constexpr int kBatch = KPO == 1 && MG == 7 ? 8 : 4;
  static_assert(G == 1 || KPO == 1, "several offsets share one k-step");
  extern __shared__ __align__(16) unsigned char smem[];
  u32x4* sw = reinterpret_cast<u32x4*>(smem);  // [step][k-step][tile][lane]
  __shared__ int s_bad;
  const int steps = (g.K3 + G - 1) / G;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, sub = lane >> 4;
  uint32_t* list = reinterpret_cast<uint32_t*>(smem + (size_t)steps * KPO * NT * 1024) + wave * (kOffsetGroup * 16);

  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.x), 0, (int)g.x_bytes, 0x00020000);

  // Blocks of 16 sorted outputs; each die (workgroups go to the eight dies in turn)
  // takes a contiguous range, whose blocks share input rows in its L2.
  const int blocks = (g.n_out + 15) / 16;
  const int per = (blocks + 7) / 8;
  const int first = ((int)blockIdx.x & 7) * per;
  const int last = min(first + per, blocks);
  const int bstride = ((int)gridDim.x >> 3) * kConvWaves;
  const int b0 = first + wave * ((int)gridDim.x >> 3) + ((int)blockIdx.x >> 3);  // small clouds use all workgroups

  // Units: (block, group of 28 offsets, 8 for K <= 2).  A unit's table entries are requested two
  // units ahead, their pairs' input rows one ahead.
  const int groups = (g.K3 + kOffsetGroup - 1) / kOffsetGroup;
  auto table = [&](int blk, int grp, int32_t* e) {
    const int p = min(blk * 16 + col, g.n_out - 1);
    const bool row = blk < last && blk * 16 + col < g.n_out;
#pragma unroll
    for (int m = 0; m < MG; ++m) {
      const int k = grp * kOffsetGroup + 4 * m + sub;
      const bool in = row && k < g.K3;
      uint32_t none = in ? 0u : 0xFFFFFFFFu;
      asm("" : "+v"(none));
      e[m] = g.omt[in ? (int64_t)k * g.stride + p : 0] | (int32_t)none;
    }
  };
  auto rows_of = [&](const int32_t* e, uint32_t* src) {
#pragma unroll
    for (int m = 0; m < MG; ++m) {
      const uint32_t r = (uint32_t)g.pin[max(e[m], 0)] * g.row_bytes;
      src[m] = e[m] >= 0 ? r : kNoRow;
    }
  };
  int32_t e[MG];
  uint32_t src[MG];
  int nb = b0, ng = 0;  // the unit whose table entries come next
  auto advance = [&]() {
    if (++ng == groups) {
      ng = 0;
      nb += bstride;
    }
  };
  table(nb, ng, e);
  advance();

  // Stage the weights; a thread moves E channels x E columns at a time.  The first
  // piece's loads, the first unit's rows and the second unit's entries go out together.
  u32x4 top = u32x4{0, 0, 0, 0};  // largest magnitudes, as bits
  {
    const T* w = static_cast<const T*>(g.w);
    constexpr int cg = KPO * SPO, cn = NT * 16 / E;
    const int pieces = steps * G * cg * cn;
    uint4 in[E];
    auto load = [&](int i) {
      const int n0 = i % cn * E, c = i / cn % cg, k = i / cn / cg;
      const bool has = i < pieces && k < g.K3 && c * E < g.c_in;
#pragma unroll
      for (int j = 0; j < E; ++j)
        in[j] = has ? *reinterpret_cast<const uint4*>(w + ((int64_t)k * g.c_in + c * E + j) * g.c_out + n0)
                    : make_uint4(0, 0, 0, 0);
    };
    auto store = [&](int i) {
      if (i >= pieces) return;
      const int n0 = i % cn * E, c = i / cn % cg, k = i / cn / cg;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const u32x4 v = __builtin_bit_cast(u32x4, in[j]) & Finite<T>::kAbs;
        if constexpr (sizeof(T) == 4)
          top = __builtin_elementwise_max(top, v);
        else
          top = __builtin_bit_cast(u32x4, __builtin_elementwise_max(__builtin_bit_cast(u16x8, top), __builtin_bit_cast(u16x8, v)));
      }
      const int step = k / G, q = G == 1 ? c / 4 : 0, sb = G == 1 ? c % 4 : k % G * SPO + c;
#pragma unroll
      for (int m = 0; m < E; ++m) {
        const int p = n0 + m;
        int t = p / 16, n = p % 16;
        if (sizeof(T) == 2 && t < (NT & ~1)) {  // inverse of conv_channel
          t = 2 * (p / 32) + (p / 4 & 1);
          n = 4 * (p / 8 % 4) + p % 4;
        }
        T out[E];
#pragma unroll
        for (int j = 0; j < E; ++j) out[j] = reinterpret_cast<const T*>(&in[j])[m];
        sw[((step * KPO + q) * NT + t) * 64 + sb * 16 + n] = *reinterpret_cast<const u32x4*>(out);
      }
    };
    load(tid);
    if (MG < 7) {
      rows_of(e, src);
      table(nb, ng, e);
      advance();
    }
    if (tid == 0) s_bad = 0;
    store(tid);
    for (int i = tid + kConvThreads; i < pieces; i += kConvThreads) {
      load(i);
      store(i);
    }
  }
  if (MG == 7) {
    rows_of(e, src);
    table(nb, ng, e);
    advance();
  }
  __syncthreads();  // (s_bad is clear)
  if (__ballot(Finite<T>::exceeded(top)) != 0 && lane == 0) s_bad = 1;
  __syncthreads();
  // A row without a pair would multiply a weight that is not finite by zero: then each
  // offset's products are summed by themselves and added to the rows that have a pair.
  const bool bad = __builtin_amdgcn_readfirstlane(s_bad) != 0;

  T* y = static_cast<T*>(g.y);
  const T* res = static_cast<const T*>(g.residual);
  const uint32_t piece = sub % SPO * 16;  // this lane's piece of an offset's channels
  uint32_t qoff[KPO];
#pragma unroll
  for (int q = 0; q < KPO; ++q) qoff[q] = (q * 4 + (G == 1 ? sub : sub % SPO)) * E < g.c_in ? q * 64 + (G == 1 ? sub * 16 : piece) : kNoRow;

  // src's rows to the list, and the steps that have any
  auto listed = [&]() {
    uint32_t todo = 0;
#pragma unroll
    for (int m = 0; m < MG; ++m) {
      list[64 * m + lane] = src[m];
      const uint64_t b = __ballot(src[m] != kNoRow);
      if constexpr (G == 4) {
        todo |= b ? 1u << m : 0u;
      } else if constexpr (G == 2) {
        todo |= ((uint32_t)b ? 1u << (2 * m) : 0u) | ((uint32_t)(b >> 32) ? 2u << (2 * m) : 0u);
      } else {
        todo |= ((uint32_t)b & 0xFFFFu ? 1u << (4 * m) : 0u) | ((uint32_t)b >> 16 ? 2u << (4 * m) : 0u) |
                ((uint32_t)(b >> 32) & 0xFFFFu ? 4u << (4 * m) : 0u) | (b >> 48 ? 8u << (4 * m) : 0u);
      }
    }
    asm volatile("" ::: "memory");
    return todo;
  };
  auto row_of = [&](int blk) {
    const int p = min(blk * 16 + col, g.n_out - 1);
    return g.perm ? (int64_t)g.perm[p] : (int64_t)p;
  };
  // each lane holds, for its row, columns 4 sub .. + 3 of every tile.  Plain stores: a
  // store writes 64 bytes of each of 16 rows, parts of lines that the caches
  // gather; non-temporal ones took 300k rows, K = 1, 48 -> 128 from 26.7 to 31.4 us, over 148
  // layers with outputs of 64 MiB and more 1.11 times as long.
  auto finish = [&](int blk, int64_t row, const f32x4* acc) {
    if (blk * 16 + col < g.n_out) {
      constexpr int W = Out<T>::N;  // channels per 16-byte vector
      constexpr int TV = W / 4;     // tiles per vector
      const int64_t at = row * g.c_out;
#pragma unroll
      for (int v = 0; v < NT / TV; ++v) {
        const int64_t o = at + conv_channel<T>(NT, v * TV, 4 * sub);
        float s[W];
#pragma unroll
        for (int t = 0; t < TV; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) s[4 * t + i] = acc[v * TV + t][i];
        if (res) Out<T>::add(s, *reinterpret_cast<const u32x4*>(res + o));
        if (g.relu) {
#pragma unroll
          for (int i = 0; i < W; ++i) s[i] = fmaxf(s[i], 0.f);
        }
        *reinterpret_cast<uint4*>(y + o) = Out<T>::pack(s);
      }
      if constexpr (NT % TV != 0) {  // the last tile of an odd count: 4 channels, 8 bytes
        const int64_t o = at + 16 * (NT - 1) + 4 * sub;
        float s[W];
#pragma unroll
        for (int i = 0; i < W; ++i) s[i] = i < 4 ? acc[NT - 1][i] : 0.f;
        if (res) {
          const uint2 rv = *reinterpret_cast<const uint2*>(res + o);
          Out<T>::add(s, u32x4{rv.x, rv.y, 0, 0});
        }
        if (g.relu) {
#pragma unroll
          for (int i = 0; i < 4; ++i) s[i] = fmaxf(s[i], 0.f);
        }
        const uint4 out = Out<T>::pack(s);
        *reinterpret_cast<uint2*>(y + o) = make_uint2(out.x, out.y);
      }
    }
  };

  if (bad) {
    for (int blk = b0; blk < last; blk += bstride) {
      f32x4 acc[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int grp = 0; grp < groups; ++grp) {
        table(blk, grp, e);
        rows_of(e, src);
        for (uint32_t todo = listed(); todo; todo &= todo - 1) {
          const int s = __builtin_ctz(todo);
          const u32x4* wp = sw + (grp * (kOffsetGroup / G) + s) * (KPO * NT * 64) + lane;
#pragma nounroll
          for (int o = 0; o < G; ++o) {
            // the step's o-th offset; zeros in the other offsets' lanes of both operands
            const uint32_t off = list[(s * G + o) * 16 + col];
            const uint32_t mine = sub / SPO == o ? 0xFFFFFFFFu : 0u;
            u32x4 a[KPO];
#pragma unroll
            for (int q = 0; q < KPO; ++q) {
              const uint32_t at = (off == kNoRow || qoff[q] == kNoRow) ? kNoRow : off + qoff[q];
              a[q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)at, 0, 0)) & mine;
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
              asm volatile("" ::: "memory");  // one tile's weights at a time (all ahead they spill)
              f32x4 part = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int q = 0; q < KPO; ++q) part = M::mma(wp[(q * NT + t) * 64] & mine, a[q], part);
#pragma unroll
              for (int j = 0; j < 4; ++j) acc[t][j] += off != kNoRow ? part[j] : 0.f;
            }
          }
        }
      }
      finish(blk, row_of(blk), acc);
    }
    return;
  }

  for (int blk = b0; blk < last; blk += bstride) {
    f32x4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int64_t row = row_of(blk);
    for (int grp = 0; grp < groups; ++grp) {
      uint32_t todo = listed();
      rows_of(e, src);  // of the next unit
      table(nb, ng, e);
      advance();
      while (todo) {
        int s[kBatch];
        u32x4 a[kBatch][KPO];
        uint32_t off[kBatch];
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
          const bool live = todo != 0;
          s[i] = live ? __builtin_ctz(todo) : 0;
          cnt += live ? 1 : 0;
          todo &= todo - 1;
          off[i] = list[(s[i] * G + sub / SPO) * 16 + col];
          if (!live) off[i] = kNoRow;
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
#pragma unroll
          for (int q = 0; q < KPO; ++q) {
            const uint32_t o = (off[i] == kNoRow || qoff[q] == kNoRow) ? kNoRow : off[i] + qoff[q];
            a[i][q] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, (int)o, 0, 0));
          }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
          if (i < cnt) {
            const u32x4* wp = sw + (grp * (kOffsetGroup / G) + s[i]) * (KPO * NT * 64) + lane;
            if constexpr (sizeof(T) == 4) {
              // a step's sum by itself: one chain over all offsets' channels rounds more.
              // Error against 64 bits, one chain -> this, and time: 60k LiDAR 32 -> 32 2.4e-7
              // -> 1.1e-7, 19.1 -> 18.9 us; 16 -> 64 1.7e-7 -> 0.9e-7, 19.5 -> 20.2 us; K = 5
              // 8 -> 32 2.0e-7 -> 0.9e-7, 30.1 -> 31.0 us (the separate steps: 1.1e-7 and 25.2
              // us, 0.9e-7 and 31.6 us, 0.9e-7 and 47.8 us).
#pragma unroll
              for (int t = 0; t < NT; ++t) {
                f32x4 part = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int q = 0; q < KPO; ++q) part = M::mma(wp[(q * NT + t) * 64], a[i][q], part);
                acc[t] += part;
              }
            } else {
#pragma unroll
              for (int q = 0; q < KPO; ++q)
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = M::mma(wp[(q * NT + t) * 64], a[i][q], acc[t]);
            }
          }
        }
      }
    }
    finish(blk, row, acc);
  }
}

struct ConvShape {
  const void* fn = nullptr;
  size_t lds = 0;
};

constexpr size_t kConvLdsMax = 160 * 1024 - 64;

// Widths and offsets that an instance serves (the reasons stand with the rule below).
constexpr bool conv_fits(int elem, int K3, int nt, int kpo, int g, int mg) {
  return kpo <= 2 * nt && (elem == 2 || K3 == 1 || kpo * nt <= 4) && conv_lds(K3, nt, kpo, g, mg) <= kConvLdsMax;
}

template <typename T, int MG>
ConvShape conv_shape_t(int K3, int nt, int kpo, int gr) {
  constexpr int kLeast = MG == 2 ? 1 : 27;  // the fewest offsets with this many entries per lane
  if (!conv_fits((int)sizeof(T), K3, nt, kpo, gr, MG)) return ConvShape{};
#define SPC_V(N, Q, G_)                                                   \
  if constexpr (conv_fits((int)sizeof(T), kLeast, N, Q, G_, MG))          \
    if (nt == N && kpo == Q && gr == G_)                                  \
      return ConvShape{reinterpret_cast<const void*>(&k_conv_small<T, N, Q, G_, MG>), conv_lds(K3, nt, kpo, gr, MG)};
#define SPC_VN(N) SPC_V(N, 1, 1) SPC_V(N, 1, 2) SPC_V(N, 1, 4) SPC_V(N, 2, 1) SPC_V(N, 3, 1) SPC_V(N, 4, 1)
  SPC_VN(1) SPC_VN(2) SPC_VN(3) SPC_VN(4) SPC_VN(6) SPC_VN(8)
#undef SPC_VN
#undef SPC_V
  return ConvShape{};
}

template <typename T>
ConvShape conv_shape_k(int K3, int nt, int kpo, int gr) {
  return K3 <= 8 ? conv_shape_t<T, 2>(K3, nt, kpo, gr) : conv_shape_t<T, 7>(K3, nt, kpo, gr);
}

// Which layers.  kpo k-steps of 64 bytes of input channels per offset (narrower inputs put
// two or four offsets into one), nt tiles of 16 output channels:
//  * the K^3 weight matrices, c_in padded to whole k-steps, fit the LDS beside the row lists:
//    16-bit K = 3: kpo * nt <= 4 (32 -> 64, 64 -> 32); 16 -> 128; K = 2: 96 -> 96, 64 -> 128;
//    K = 5: 32 -> 16, 16 -> 32, 8 -> 64;
//  * kpo <= 2 nt (each block's input rows are requested once per offset whatever the
//    width: 128 -> 16, K = 3, 183k voxels took 48.4 us against the separate steps' 43.2;
//    48 and 64 -> 16, K = 3: 0.77 times their time over 60 layers).  K = 1 in 16 bits and widths
//    that the centre scatter takes, one launch as well: kpo < 2 nt (128 -> 32, 179k voxels
//    15.2 against 14.3 us);
//  * 16 bits, K = 2 or 3, under 512 blocks and 3.1 pairs per output: at most 64 KiB of
//    weights, which every workgroup stages (500 voxels, K = 3, 32 -> 64 9.4 against 7.9 us,
//    K = 2, 64 -> 128 8.9 against 6.5; 54 KiB, K = 3, 32 -> 32, never over 1.02; with 7.4 pairs
//    per output 32 -> 64 never; K = 5, 32 -> 16 15.3 against 28.0: one offset's rows fill no
//    tile of the separate steps, in two launches);
//  * float32 (K > 1): kpo * nt <= 4, 2 under 512 blocks.  A block's products run in one
//    wave, at every offset that any of its rows lists, and float32 MFMAs take twice the
//    cycles for an eighth of the work: 64 -> 64, K = 2, 86k voxels 37.5 against 34.6 us.
//    For K = 3 the separate steps, which multiply listed pairs only, win where few of a
//    block's rows share an offset.  Under 3.1 pairs per output: kpo = 1 (32 -> 32, 120k LiDAR
//    voxels 38.2 against 32.7 us, room down 70.9 against 51.7; at 5.6 pairs, 30k LiDAR 13.5
//    against 22.9); under 512 blocks nt = 1 (16 -> 32, 2k voxels 9.1 against 8.3 us), or 2
//    with four offsets per step; and under 1.18 pairs kpo * nt <= 3 (scattered voxels, stride
//    2, 16 -> 64 35.4 against 30.8 us; at 1.2 pairs, stride 1, 24.9 against 31.4).
ConvShape conv_shape(int64_t n_out, int64_t pairs, int K3, int c_in, int c_out, int dtype) {
  if (c_out % 16 != 0) return ConvShape{};
  const int ks = dtype == 0 ? 16 : 32;  // channels per k-step
  const int gr = c_in * 4 <= ks ? 4 : (c_in * 2 <= ks ? 2 : 1);
  const int kpo = gr > 1 ? 1 : (c_in + ks - 1) / ks;
  if (gr > 1 && c_in * gr != ks) return ConvShape{};
  const int nt = c_out / 16;
  const bool few = n_out < 512 * 16, sparse = 10 * pairs < 31 * n_out;
  if (dtype != 0) {
    if (K3 == 1 && c_out % 32 == 0 && kpo >= 2 * nt) return ConvShape{};
    if (K3 > 1 && K3 <= 27 && few && sparse && (K3 + gr - 1) / gr * kpo * nt > 64) return ConvShape{};
  } else if (K3 > 1) {
    if (few && kpo * nt > 2) return ConvShape{};
    if (K3 == 27 && sparse &&
        (kpo > 1 || (few && nt > 1 && gr < 4) || (kpo * nt == 4 && gr == 1 && 50 * pairs < 59 * n_out)))
      return ConvShape{};
  }
  if (dtype == 0) return conv_shape_k<float>(K3, nt, kpo, gr);
  if (dtype == 1) return conv_shape_k<__half>(K3, nt, kpo, gr);
  return conv_shape_k<__hip_bfloat16>(K3, nt, kpo, gr);
}

// (positions up to two rounds of blocks past the last output are held in 32 bits)
bool conv_rows_fit(int64_t n_in, int64_t n_out, int c_in, int dtype) {
  return n_out < ((int64_t)1 << 31) - (1 << 16) && n_in * c_in * (dtype == 0 ? 4 : 2) <= kMaxInputBytes;
}

}  // namespace

bool conv_small_applies(int64_t n_in, int64_t n_out, int64_t pairs, int K3, int c_in, int c_out, int dtype) {
  return conv_rows_fit(n_in, n_out, c_in, dtype) && conv_shape(n_out, pairs, K3, c_in, c_out, dtype).fn;
}

hipError_t launch_conv_small(const void* x, int64_t n_in, const void* w, const int32_t* pin, const int32_t* omt,
                             int64_t mt_stride, const uint32_t* perm, int64_t pairs, int K3, void* y,
                             const void* residual, int relu, int64_t n_out, int c_in, int c_out, int dtype,
                             hipStream_t s) {
  if (n_out <= 0) return hipSuccess;
  const ConvShape sh = conv_shape(n_out, pairs, K3, c_in, c_out, dtype);
  if (!sh.fn || !conv_rows_fit(n_in, n_out, c_in, dtype)) return hipErrorInvalidValue;
  ProfScope ps(KN_CONV_SMALL, s);
  ConvArgs g;
  g.x = x;
  g.w = w;
  g.pin = pin;
  g.omt = omt;
  g.stride = mt_stride;
  g.perm = perm;
  g.y = y;
  g.residual = residual;
  g.K3 = K3;
  g.n_out = (int)n_out;
  g.c_in = c_in;
  g.c_out = c_out;
  g.relu = relu;
  g.row_bytes = (uint32_t)(c_in * (dtype == 0 ? 4 : 2));
  g.x_bytes = (uint32_t)n_in * g.row_bytes;
  // one workgroup per CU, about four blocks per workgroup on small clouds; a multiple of
  // eight, one share of the blocks per die
  const int64_t blocks = (n_out + 15) / 16;
  const unsigned grid = (unsigned)std::min<int64_t>(256, ((blocks + 3) / 4 + 7) / 8 * 8);
  void* args[] = {&g};
  return hipLaunchKernel(sh.fn, dim3(grid), dim3(kConvThreads), args, sh.lds, s);
}

}  // namespace spc
