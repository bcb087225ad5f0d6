// The convolutions proper: dense contractions on CDNA4 matrix cores (MFMA).
//
// A sparse convolution (Section 2.3) computes, for every active output row o
// and for the ground row, b + sum_f W_f^T x_{R[o][f]}: a GEMM whose A operand
// is gathered row by row through the window lists.  The gather is fused into
// the LDS fill of the A tile (no gathered matrix is written to HBM); weights
// are packed once per step into [N][K] tiles and staged through LDS.
//
//  * forward      out = ReLU(G W + b)        rows: output sites + ground row
//  * input grad   dX  = sum_f delta[Rt[.][f]] W_f^T   rows: sites below
//  * softmax head logits = h W + b, dh = dlogits W^T  (window of one)
//  * weight grad  dW = G^T delta, split over sites (for the softmax layer one
//                 extra A row of ones also gives db = sum delta).
//
// bf16: v_mfma_f32_16x16x32_bf16 (one per 32-wide k block);
// fp32: v_mfma_f32_16x16x4f32 (four per 16-wide k block).  Accumulation is
// always fp32.

#include "common.h"
#include "epilogue.h"
#include "pool_route.h"
#include "ground_tasks.h"
#include "kernels.h"

#include <hip/hip_ext.h>

#include <type_traits>

namespace sscn {

template <typename T>
struct MfmaCore;

template <>
struct MfmaCore<__bf16> {
  static constexpr int KB = 32;  // k per block
  __device__ static inline void step(const __bf16* a_ptr, const __bf16* b_ptr, f32x4& acc) {
    bf16x8 a = *(const bf16x8*)a_ptr;
    bf16x8 b = *(const bf16x8*)b_ptr;
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
  }
};

template <>
struct MfmaCore<float> {
  static constexpr int KB = 16;  // four 16x16x4 steps: step e takes k = 4 g + e of lane group g on both sides
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Tile configuration: WM x WN waves, each computing TM x TN 16x16 MFMA tiles;
// K advances in slabs of 128 bytes per row (64 bf16 / 32 fp32 elements).
template <typename T, int WM_, int WN_, int TM_, int TN_>
struct GCfg {
  static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_;
  static constexpr int NT = 64 * WM * WN;
  static constexpr int BM = WM * TM * 16, BN = WN * TN * 16;
  static constexpr int VE = Elem<T>::VE;
  static constexpr int KB = MfmaCore<T>::KB;
  static constexpr int BK = 2 * KB;
  static constexpr int KV = BK / VE;       // 16-byte vectors per row and slab
  static constexpr int AV = BM * KV / NT;  // A vectors per thread and slab
  static constexpr int BV = BN * KV / NT;
  static_assert(AV * NT == BM * KV && BV * NT == BN * KV, "tile must split evenly over the threads");
  // first column of the tile that wave column wn's block j computes: the waves'
  // blocks interleave, so that where the columns end inside a tile its waves
  // are left with equal numbers of live blocks
  __device__ static inline int col(int wn, int j) { return (j * WN + wn) * 16; }
  // the weight gradients' rows likewise
  __device__ static inline int row(int wm, int i) { return (i * WM + wm) * 16; }
};

constexpr int AMAX = 9;  // largest window (3x3)

// the four tile shapes (index = GemmArgs::cfg)
// (bf16 multiplies square wave tiles, whose operands take the fewest LDS reads;
// float32, whose MFMAs outlast them, gives every wave whole rows, so that dead
// column blocks leave all waves alike; its 32 x 64 tile, with rows for two waves
// only, keeps two columns of waves, and with one live block the second multiplies a
// dead one)
template <typename T> using C128x128 = GCfg<T, sizeof(T) == 2 ? 2 : 4, sizeof(T) == 2 ? 2 : 1, sizeof(T) == 2 ? 4 : 2, sizeof(T) == 2 ? 4 : 8>;
template <typename T> using C128x64 = GCfg<T, 4, 1, 2, 4>;
template <typename T> using C64x64 = GCfg<T, sizeof(T) == 2 ? 2 : 4, sizeof(T) == 2 ? 2 : 1, sizeof(T) == 2 ? 2 : 1, sizeof(T) == 2 ? 2 : 4>;
template <typename T> using C32x64 = GCfg<T, 2, 2, 1, 2>;

int gemm_bm(bool bf16, int cfg) { return cfg == GEMM_DIRECT ? DIRECT_BM : gemm_tile(bf16, cfg).BM; }

GemmTile gemm_tile(bool bf16, int cfg) {
  const int BK = bf16 ? 64 : 32;
  switch (cfg) {
    case 0: return GemmTile{128, 128, BK};
    case 1: return GemmTile{128, 64, BK};
    case 2: return GemmTile{64, 64, BK};
    default: return GemmTile{32, 64, BK};
  }
}

// acc[i][j] += A_tile(wave rows i) * B_tile(wave column blocks j) over one slab
// held in LDS unpadded and swizzled: row r's 16-byte chunk c sits in slot
// c ^ ((r / 2) % 8) of its 128-byte row, so the sixteen rows an MFMA operand
// read touches cover all 64 banks once.  Only the wave's first LIVE column
// blocks are computed.
template <typename T, class C, int LIVE>
__device__ inline void mma_slab(const T* As, const T* Bs, f32x4 (&acc)[C::TM][C::TN], int wm, int wn, int lane) {
  constexpr int VE = C::VE;
  const int r16 = lane & 15, g = lane >> 4;
  auto a_at = [&](int i, int chunk) {
    const int r = wm * C::TM * 16 + i * 16 + r16;
    return As + r * C::BK + ((chunk ^ ((r >> 1) & 7)) * VE);
  };
  auto b_at = [&](int j, int chunk) {
    const int r = C::col(wn, j) + r16;
    return Bs + r * C::BK + ((chunk ^ ((r >> 1) & 7)) * VE);
  };
#pragma unroll
  for (int kb = 0; kb < C::BK; kb += C::KB) {
    const int chunk = kb / VE + g;
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < LIVE; ++j) MfmaCore<T>::step(a_at(i, chunk), b_at(j, chunk), acc[i][j]);
    } else {
      f32x4 av[C::TM], bv[LIVE];
#pragma unroll
      for (int i = 0; i < C::TM; ++i) av[i] = *(const f32x4*)a_at(i, chunk);
#pragma unroll
      for (int j = 0; j < LIVE; ++j) bv[j] = *(const f32x4*)b_at(j, chunk);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < LIVE; ++j)
#pragma unroll
          for (int i = 0; i < C::TM; ++i)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i][e], bv[j][e], acc[i][j], 0, 0, 0);
    }
  }
}

// Calls run(integral_constant<int, N>) with the smallest N in [LO, HI] that is at
// least n (HI when none is).
template <int LO, int HI, class F>
__device__ inline void with_count(int n, F&& run) {
  if constexpr (LO < HI) {
    if (n > LO) {
      with_count<LO + 1, HI>(n, run);
      return;
    }
  }
  run(std::integral_constant<int, LO>{});
}

// s_waitcnt vmcnt(n) lgkmcnt(0), n a compile-time constant: the LDS reads of
// the previous slab are done before its stage is refilled
template <int N>
__device__ inline void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt field");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));  // lgkmcnt(0) too
}

// One 16-byte load per lane from a buffer straight into LDS: lane l's bytes
// land at LDS byte address lds + 16 l (lds uniform over the wave). An offset
// at or past the buffer's size reads zero. The compiler does not see this
// load, so the caller waits for it with wait_vmcnt; its own waits only grow
// stricter with loads it does not know of. No memory clobber: the caller
// orders the load against the LDS reads of the same stage with compiler
// fences around its barriers.
__device__ inline void dma16(u32x4 rsrc, uint32_t lds, uint32_t off) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds),
      "v"(off), "s"(rsrc)
      : "m0");
}

// The same for 4 bytes per lane: lane l's dword lands at lds + 4 l.
__device__ inline void dma4(u32x4 rsrc, uint32_t lds, uint32_t off) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "buffer_load_dword %1, %2, 0 offen lds" ::"s"(lds),
      "v"(off), "s"(rsrc)
      : "m0");
}

// The same two loads from a 64-bit address per lane (float32: its feature
// arrays may pass the 2 GiB that a buffer's offsets reach; a lane without a
// source reads zeros from an address that holds them).
__device__ inline void dma16_at(uint32_t lds, const void* p) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off" ::"s"(lds),
      "v"(p)
      : "m0");
}
__device__ inline void dma4_at(uint32_t lds, const void* p) {
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dword %1, off" ::"s"(lds),
      "v"(p)
      : "m0");
}

// raw buffer descriptor: base, no stride, size in bytes
__device__ inline u32x4 buffer_rsrc(const void* base, uint32_t bytes) {
  const uint64_t b = (uint64_t)base;
  return u32x4{(uint32_t)b, (uint32_t)(b >> 32) & 0xffffu, bytes, 0x00020000u};
}

__device__ inline uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// q = k / d for 0 <= k < 2^20, 1 <= d < 2^16: float estimate, then exact correction.
__device__ inline int div_small(int k, int d, float rcp) {
  int q = (int)((float)k * rcp);
  q += (q + 1) * d <= k ? 1 : 0;
  q -= q * d > k ? 1 : 0;
  return q;
}

// Routing inputs of the items a thread takes in store_staged (AC >= 0 and at
// most two items per thread, four of float32's half as wide ones), all loaded
// before the first item is routed: one memory round trip for the thread's
// items, not one each.
template <typename T, class C, int AC>
struct StagedRoute {
  static constexpr int NV = C::BN / C::VE;
  static constexpr int IPT = (C::BM * NV + C::NT - 1) / C::NT;  // items per thread
  static constexpr bool ON = AC >= 0 && IPT <= (sizeof(T) == 2 ? 2 : 4);
  RouteIn<T, AC < 0 ? 0 : AC> q[ON ? IPT : 1];
  __device__ inline void load(const GemmArgs& a, int m0, int n0, int rows) {
    if constexpr (ON) {
#pragma unroll
      for (int i = 0; i < IPT; ++i) {
        const int v = threadIdx.x + i * C::NT;
        const int r = v / NV, m = m0 + r, n = n0 + (v - r * NV) * C::VE;
        if (v < C::BM * NV && m >= 1 && m < rows && n < a.out_cols)
          route_load_window<T, AC < 0 ? 0 : AC>(a.pr, m, n, q[i]);
      }
    }
  }
};

// Stores of an output tile staged in LDS (Cs, pitch CS), 16 bytes at a time.
// AC >= 0: the pooling backward of every row m >= 1 as well, and the tile's
// slot partial sums as partial tm (lds: the staging buffer, reused; LDSF floats).
template <typename T, class C, int CS, int AC, int LDSF>
__device__ inline void store_staged(const GemmArgs& a, const T* Cs, int m0, int n0, int tm, int rows, float* lds) {
  constexpr int VE = C::VE, BM = C::BM, BN = C::BN, NT = C::NT, NV = BN / VE;
  constexpr bool SUMS = AC == MASK_MODE;  // the column sums of the rows stored (GemmArgs::sums)
  constexpr int J = AC >= 0 ? 2 + AC : 1;
  static_assert(NT % NV == 0, "each thread keeps one channel vector");
  float acc[J][VE];
  if constexpr (AC >= 0 || SUMS) {
#pragma unroll
    for (int k = 0; k < J; ++k)
#pragma unroll
      for (int e = 0; e < VE; ++e) acc[k][e] = 0.f;
  }
  if constexpr (StagedRoute<T, C, AC>::ON) {
    StagedRoute<T, C, AC> pre;
    pre.load(a, m0, n0, rows);
#pragma unroll
    for (int i = 0; i < StagedRoute<T, C, AC>::IPT; ++i) {
      const int v = threadIdx.x + i * NT;
      const int r = v / NV, nv = v - r * NV;
      const int m = m0 + r, n = n0 + nv * VE;
      if (v < BM * NV && m < rows && n < a.out_cols) {
        const u32x4 o = *(const u32x4*)(Cs + r * CS + nv * VE);
        *(u32x4*)((T*)a.out + (int64_t)m * a.out_stride + n) = o;
        if (m >= 1) {
          route_load_children<T, AC>(a.pr, n, pre.q[i]);
          route_apply<T, AC>(a.pr, n, pre.q[i], (const T*)&o, acc);
        }
      }
    }
  } else {
    for (int v = threadIdx.x; v < BM * NV; v += NT) {
      const int r = v / NV, nv = v - r * NV;
      const int m = m0 + r, n = n0 + nv * VE;
      if (m < rows && n < a.out_cols) {
        const u32x4 o = *(const u32x4*)(Cs + r * CS + nv * VE);
        *(u32x4*)((T*)a.out + (int64_t)m * a.out_stride + n) = o;
        if constexpr (AC >= 0)
          if (m >= 1) pool_route_item<T, AC>(a.pr, m, n, (const T*)&o, acc);
        if constexpr (SUMS) {
#pragma unroll
          for (int e = 0; e < VE; ++e) acc[0][e] += Elem<T>::to_f32(((const T*)&o)[e]);
        }
      }
    }
  }
  if constexpr (SUMS)
    if (a.sums) tile_slot_sums<VE, J, NT, NV, LDSF>(acc, lds, a.pr, n0, tm, 1);
  if constexpr (AC >= 0) tile_slot_sums<VE, J, NT, NV, LDSF>(acc, lds, a.pr, n0, tm);
}

// Pooling forward in the epilogue (GemmArgs::pool_fwd): the staged tile's
// rows are the slots 4 p + f of pooling windows p (m0 is a multiple of 4).
// Every slot's convolution row Cr is stored (row 0 from slot 0 only: the
// ground value), then each window's first maximum over its four slots, per
// channel, goes to the pooling layer with its position.
template <typename T, class C, int CS>
__device__ inline void store_pooled(const GemmArgs& a, const T* Cs, const int32_t* Cr, int m0, int n0, int rows) {
  constexpr int VE = C::VE, BM = C::BM, BN = C::BN, NT = C::NT, NV = BN / VE;
  typedef typename ArgPack<VE>::W AW;
  static_assert(BM % 4 == 0, "whole windows per tile");
  for (int v = threadIdx.x; v < BM * NV; v += NT) {
    const int r = v / NV, nv = v - r * NV;
    const int m = m0 + r, n = n0 + nv * VE;
    const int row = Cr[r];
    if (m < rows && n < a.out_cols && (row > 0 || m == 0))
      *(u32x4*)((T*)a.out + (int64_t)row * a.out_stride + n) = *(const u32x4*)(Cs + r * CS + nv * VE);
  }
  for (int v = threadIdx.x; v < (BM / 4) * NV; v += NT) {
    const int pr = v / NV, nv = v - pr * NV;
    const int m = m0 + 4 * pr, n = n0 + nv * VE;
    if (m >= rows || n >= a.out_cols) continue;
    // running first maximum over the four slots (one staged vector at a time)
    u32x4 out = *(const u32x4*)(Cs + (4 * pr) * CS + nv * VE);
    AW am = 0;
#pragma unroll
    for (int f = 1; f < 4; ++f) {
      const u32x4 in = *(const u32x4*)(Cs + (4 * pr + f) * CS + nv * VE);
#pragma unroll
      for (int j = 0; j < VE; ++j) {
        const bool gt = Elem<T>::to_f32(((const T*)&in)[j]) > Elem<T>::to_f32(((const T*)&out)[j]);
        if (gt) {
          ((T*)&out)[j] = ((const T*)&in)[j];
          am = (am & ~((AW)0xff << (8 * j))) | ((AW)f << (8 * j));
        }
      }
    }
    const int64_t p = m / 4;
    *(u32x4*)((T*)a.pool_out + p * a.pool_stride + n) = out;
    *(AW*)(a.pool_argmax + p * a.pool_stride + n) = am;
  }
}

// Row offset of a window entry that names no row: at or past the end of the
// source buffer whatever channel is added, so its loads read zero.
constexpr uint32_t GATHER_NONE = 0x80000000u;

// Chunk c (8 k) of the bf16 GEMM's K: its window position (bits 27..30), its
// channel's byte offset in the source row (bits 0..26), and GATHER_NONE past K.
// Looked up per slab instead of divided out: the slab's loads took 45 VALU
// instructions a thread, a third of all the tile's, against 15.
__device__ inline int chunk_word(const GemmArgs& a, int c, float rcp_cseg) {
  const int k = c * 8;
  if (k >= a.K) return (int)GATHER_NONE;
  if (a.A == 1) return k * 2;
  const int f = div_small(k, a.cseg, rcp_cseg);
  return f << 27 | (k - f * a.cseg) * 2;
}

// Implicit-gather GEMM.  Per tile: the tile's window rows go to LDS once; the
// K slabs stream through a ring of LDS stages filled by loads with an LDS
// destination (bf16: buffer loads, an offset past the buffer reads zero;
// float32: loads from 64-bit addresses); the output tile is staged in LDS for
// 16-byte stores.
// With ksplit > 1 each workgroup covers one K range and writes fp32 partial
// sums, reduced (with the epilogue) by k_gemm_splitk_reduce.
template <typename T, class C, int RAC>
__global__ void __launch_bounds__(C::NT) k_gemm_gather(GemmArgs a) {
  constexpr int VE = C::VE, BK = C::BK, BM = C::BM, BN = C::BN, NT = C::NT;
  constexpr int CS = BN + VE;  // staging pitch
  constexpr bool POOL = RAC == POOL_FWD_MODE;
  // NST slabs in LDS, NST - 1 of them in flight while one is multiplied, one
  // barrier per slab.  Two stages where three would cost occupancy (the 128x128
  // tile; the pooled forward, which then fits three workgroups per compute unit
  // and its launches one round of workgroups) or measured slower (the routed
  // tiles, whose epilogue holds more registers).
  constexpr int NST = (BM + BN >= 256 || (sizeof(T) == 2 && (RAC >= 0 || POOL))) ? 2 : 3;
  constexpr int STG = (BM + BN) * BK;          // elements per stage
  constexpr int LPS = C::AV + C::BV;           // loads per thread and slab
  constexpr bool MASK = RAC == MASK_MODE;
  // the masked store stages the layer below's tile beside its own, where that leaves two workgroups a compute unit
  constexpr bool MASK_LDS = MASK && BM * (CS + BN) * (int)sizeof(T) <= 80 * 1024;
  constexpr int OUT = BM * CS + (MASK_LDS ? BM * BN : 0);
  constexpr int SMEM = NST * STG > OUT ? NST * STG : OUT;
  __shared__ __attribute__((aligned(16))) T smem[SMEM];
  // sized at launch: [BM * A] window entries (bf16: the source row's byte offset,
  // GATHER_NONE where there is none; float32: its row, -1), then (bf16, A > 1) one
  // word per 16-byte chunk of K, see chunk_word
  extern __shared__ int32_t Rs[];
  __shared__ int32_t Cr[POOL ? BM : 1];  // pooling forward: the convolution row of each slot

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / C::WN, wn = wave % C::WN;
  if (run_extra<T>(a.x)) return;
  const int rows = (a.rows_dev ? (*a.rows_dev + a.rows_add) : a.rows_host) * (POOL ? 4 : 1);
  const int span = rows - a.row_begin;
  if (span <= 0) return;
  const int tiles_m = (span + BM - 1) / BM;
  const int tiles_n = a.Npad / BN;
  const int kslabs = a.Kpad / BK;
  const int kper = (kslabs + a.ksplit - 1) / a.ksplit * BK;
  const int ntiles = tiles_m * tiles_n * a.ksplit;
  const T* src = (const T*)a.src;
  const T* Bt = (const T*)a.Bt;
  const int A = a.A;
  const float rcp_cseg = 1.f / (float)a.cseg;
  const uint32_t row_bytes = (uint32_t)a.src_stride * (uint32_t)sizeof(T);
  bool tabled = false;

  const int grid = own_grid(a.x);
  const TileDeal deal = deal_tiles(ntiles, grid, blockIdx.x, deal_by_xcd(tiles_n, a.rmap != nullptr, a.A, a.ksplit));
  for (int tile = deal.first; tile < deal.end; tile += deal.step) {
    const int tn = tile % tiles_n;
    const int t2 = tile / tiles_n;
    const int tm = t2 % tiles_m;
    const int ks = t2 / tiles_m;
    const int m0 = a.row_begin + tm * BM, n0 = tn * BN;
    const int kbeg = ks * kper;
    const int kend = min(a.Kpad, kbeg + kper);

    if (tid < BM) {  // the tile's window rows: one row per thread, all loads issued before any store
      const int m = m0 + tid;
      const bool live = m < rows;
      int row = m;  // the output row (pooling forward: the slot's convolution row)
      if constexpr (POOL) {
        const int pr = a.pslot[live ? m : 0];
        row = live ? pr : 0;
        Cr[tid] = row;
      }
      int v[AMAX];
      if (a.rmap) {  // rows past the count read row 0's window and discard it
        const int32_t* rp = a.rmap + (int64_t)(live ? row : 0) * A;
#pragma unroll
        for (int f = 0; f < AMAX; ++f) v[f] = rp[f < A ? f : 0];
      } else {
#pragma unroll
        for (int f = 0; f < AMAX; ++f) v[f] = f == 0 ? row : -1;
      }
#pragma unroll
      for (int f = 0; f < AMAX; ++f)
        if (f < A) {
          if constexpr (sizeof(T) == 2)
            Rs[tid * A + f] = live && v[f] >= 0 ? v[f] * row_bytes : (int)GATHER_NONE;
          else
            Rs[tid * A + f] = live ? v[f] : -1;
        }
    }
    if constexpr (sizeof(T) == 2)
      if (!tabled && A > 1) {  // the same for every tile
        for (int c = tid; c < a.Kpad / VE; c += NT) Rs[BM * A + c] = chunk_word(a, c, rcp_cseg);
        tabled = true;
      }
    __syncthreads();

    f32x4 acc[C::TM][C::TN];
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int j = 0; j < C::TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // The masked store's output tile of the layer below: 16-byte loads before the K
    // loop, through LDS after it.  (Loaded where they are used, two bytes a lane in
    // the MFMA result's layout: 29.4 us for the 128 x 128 tiles of DeepCNiN(5,50)'s
    // second input gradient, 19.4 like this.)
    constexpr int MV = MASK_LDS ? BM * BN / VE / NT : 1;
    u32x4 mk[MV];
    if constexpr (MASK_LDS) {
      static_assert(MV * NT * VE == BM * BN, "whole vectors per thread");
#pragma unroll
      for (int i = 0; i < MV; ++i) {
        const int v = tid + i * NT, r = v / (BN / VE), n = n0 + (v - r * (BN / VE)) * VE;
        const bool in = m0 + r < rows && n < a.out_cols;
        mk[i] = *(const u32x4*)((const T*)a.mask + (in ? (int64_t)(m0 + r) * a.mask_stride + n : 0));
      }
    }
    // this wave's column blocks below the result's width
    const int live =
        __builtin_amdgcn_readfirstlane((min(a.out_cols - n0, BN) - wn * 16 + 16 * C::WN - 1) / (16 * C::WN));
    {
      // A: one 16-byte slot per load (row v / 8, slot v % 8 holding chunk
      // (v % 8) ^ ((row / 2) % 8)); rows without a window entry and k past K read zero
      const u32x4 rsA = buffer_rsrc(src, GATHER_SRC_BYTES);
      const u32x4 rsB = buffer_rsrc(Bt, (uint32_t)a.Npad * (uint32_t)a.Kpad * 2u);
      const int wave_u = __builtin_amdgcn_readfirstlane(wave);  // in a scalar register
      const uint32_t lds0 = lds_addr(smem);
      const int chunk = (tid & 7) ^ ((tid >> 4) & 7);
      auto issue = [&](int k0, int st) {
        const uint32_t la = lds0 + (uint32_t)(st * STG * (int)sizeof(T)), lb = la + BM * BK * (int)sizeof(T);
        // (every slot of a thread holds the same chunk: one window position and
        // channel per slab)
        static_assert(NT == 256, "rows 32 apart share their swizzle");
        if constexpr (sizeof(T) == 2) {
          // (a window of one: K is the row itself, whatever its length)
          const int w = A > 1 ? Rs[BM * A + k0 / VE + chunk] : chunk_word(a, k0 / VE + chunk, rcp_cseg);
          const uint32_t col = w & ((1 << 27) - 1), none = w & GATHER_NONE;
          const int32_t* R = Rs + (tid >> 3) * A + ((w >> 27) & 0xf);
          uint32_t off[C::AV];
#pragma unroll
          for (int j = 0; j < C::AV; ++j)  // every window row read before the first load goes out
            off[j] = ((uint32_t)R[j * (NT / 8) * A] + col) | none;
#pragma unroll
          for (int j = 0; j < C::AV; ++j) dma16(rsA, la + (uint32_t)(wave_u * 64 + j * NT) * 16u, off[j]);
          const uint32_t bcol = (uint32_t)((n0 + (tid >> 3)) * a.Kpad + k0 + chunk * VE) * 2u;
#pragma unroll
          for (int j = 0; j < C::BV; ++j)
            dma16(rsB, lb + (uint32_t)(wave_u * 64 + j * NT) * 16u, bcol + (uint32_t)(j * (NT / 8) * a.Kpad) * 2u);
        } else {
          // (selects, no branches)
          const int k = k0 + chunk * VE;
          const bool in_k = k < a.K;
          const int f = div_small(k, a.cseg, rcp_cseg);
          const T* col = src + (k - f * a.cseg);
          const int32_t* R = Rs + (tid >> 3) * A + (in_k ? f : 0);
          int srow[C::AV];
#pragma unroll
          for (int j = 0; j < C::AV; ++j) srow[j] = R[j * (NT / 8) * A];
#pragma unroll
          for (int j = 0; j < C::AV; ++j) {
            const uint64_t at = (uint64_t)col + (uint64_t)(uint32_t)srow[j] * row_bytes;
            dma16_at(la + (uint32_t)(wave_u * 64 + j * NT) * 16u,
                     (const void*)(in_k && srow[j] >= 0 ? at : (uint64_t)a.zero));
          }
          const T* bcol = Bt + ((int64_t)(n0 + (tid >> 3)) * a.Kpad + k);
#pragma unroll
          for (int j = 0; j < C::BV; ++j)
            dma16_at(lb + (uint32_t)(wave_u * 64 + j * NT) * 16u, bcol + (int64_t)j * (NT / 8) * a.Kpad);
        }
      };
      const int nsl = kend > kbeg ? (kend - kbeg) / BK : 0;  // (a K range may be empty: its sums are zero)
#pragma unroll
      for (int p = 0; p < NST - 1; ++p)
        if (p < nsl) issue(kbeg + p * BK, p);
      auto slab_loop = [&](auto live_c) {
        constexpr int LIVE = decltype(live_c)::value;
        for (int s = 0; s < nsl; ++s) {
          // this wave's loads of slab s have landed once at most those of the
          // slabs after it are outstanding; the barrier makes it every wave's
          asm volatile("" ::: "memory");
          if constexpr (NST == 3) {
            if (s + 1 < nsl) wait_vmcnt<LPS>(); else wait_vmcnt<0>();
          } else {
            wait_vmcnt<0>();
          }
          __builtin_amdgcn_s_barrier();
          asm volatile("" ::: "memory");
          if (s + NST - 1 < nsl) issue(kbeg + (s + NST - 1) * BK, (s + NST - 1) % NST);
          mma_slab<T, C, LIVE>(smem + (s % NST) * STG, smem + (s % NST) * STG + BM * BK, acc, wm, wn, lane);
        }
      };
      // float32: column blocks past the result's width are not multiplied (a
      // block costs TM x 4 MFMAs of 32 cycles per 16 k), with a copy of the loop
      // for each count (branches around the MFMAs cost more than they save: the
      // 64 x 64 tile's input gradients 39 -> 59 us); bf16 multiplies them all.
      // (Every wave passes the same barriers in whichever copy it runs.)
      if constexpr (sizeof(T) == 2)
        slab_loop(std::integral_constant<int, C::TN>{});
      else
        with_count<C::TN == 8 ? 5 : 1, C::TN>(live, slab_loop);
      asm volatile("" ::: "memory");
      __syncthreads();  // every wave done with the slabs before the epilogue reuses the memory
    }

    const int g = lane >> 4, c16 = lane & 15;
    float bias[C::TN];
#pragma unroll
    for (int j = 0; j < C::TN; ++j) {
      const int n = n0 + C::col(wn, j) + c16;
      bias[j] = (a.bias && n < a.N) ? a.bias[n] : 0.f;
    }
    if (a.ksplit > 1) {
      float* part = a.part + (int64_t)ks * a.part_rows * a.Npad;
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j) {
          const int n = n0 + C::col(wn, j) + c16;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int m = m0 + wm * C::TM * 16 + i * 16 + g * 4 + r;
            if (m < rows) part[(int64_t)m * a.Npad + n] = acc[i][j][r];
          }
        }
    } else if (epi_stores_T(a.epi)) {
      T* Cs = smem;
      T* Ms = smem + BM * CS;
      if constexpr (MASK_LDS) {
#pragma unroll
        for (int i = 0; i < MV; ++i) *(u32x4*)(Ms + (tid + i * NT) * VE) = mk[i];
        __syncthreads();
      }
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j) {
          const int nl = C::col(wn, j) + c16;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int ml = wm * C::TM * 16 + i * 16 + g * 4 + r;
            // the gradients' epilogues (EPI_STORE, EPI_STORE_MASK) have no bias or rectifier
            float v = RAC >= 0 || MASK ? acc[i][j][r] : epi_value<T>(a, acc[i][j][r], bias[j]);
            if constexpr (MASK) {  // the rectifier derivative of the layer below, before the one rounding to storage
              if constexpr (MASK_LDS)
                v *= act_factor(Elem<T>::to_f32(Ms[ml * BN + nl]), a.slope);
              else if (m0 + ml < rows && n0 + nl < a.out_cols)
                v *= act_factor(
                    Elem<T>::to_f32(((const T*)a.mask)[(int64_t)(m0 + ml) * a.mask_stride + n0 + nl]), a.slope);
            }
            Cs[ml * CS + nl] = Elem<T>::from_f32(v);
          }
        }
      __syncthreads();
      if constexpr (POOL)
        store_pooled<T, C, CS>(a, Cs, Cr, m0, n0, rows);
      else
        store_staged<T, C, CS, RAC, SMEM * (int)sizeof(T) / 4>(a, Cs, m0, n0, tm, rows, (float*)smem);
    } else {
#pragma unroll
      for (int i = 0; i < C::TM; ++i)
#pragma unroll
        for (int j = 0; j < C::TN; ++j) {
          const int n = n0 + C::col(wn, j) + c16;
          if (n >= a.out_cols) continue;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int m = m0 + wm * C::TM * 16 + i * 16 + g * 4 + r;
            if (m < rows) store_out<T>(a, m, n, epi_value<T>(a, acc[i][j][r], bias[j]));
          }
        }
    }
    __syncthreads();
  }
}

// Sum of the split-K partials plus the epilogue: four consecutive columns per
// thread, one 16-byte partial load per split (the partials are Npad wide).
template <typename T>
__global__ void __launch_bounds__(256) k_gemm_splitk_reduce(GemmArgs a) {
  const int rows = a.rows_dev ? (*a.rows_dev + a.rows_add) : a.rows_host;
  const int64_t span = rows - a.row_begin;
  if (span <= 0) return;
  const int quads = (a.out_cols + 3) / 4;
  const int64_t total = span * quads;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t m = a.row_begin + t / quads;
    const int n = (int)(t % quads) * 4;
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int ks = 0; ks < a.ksplit; ++ks) s += *(const f32x4*)(a.part + ((int64_t)ks * a.part_rows + m) * a.Npad + n);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n + e < a.out_cols) store_out<T>(a, m, n + e, epi_value<T>(a, s[e], (a.bias && n + e < a.N) ? a.bias[n + e] : 0.f));
  }
}

// Site chunks of a layer (ChunkPlan; the softmax layer has one).
__device__ inline int wgrad_chunks(const WGradArgs& a) { return a.nch_dev ? *a.nch_dev : 1; }

// Layers of at least this many chunks have all tiles of a chunk on one XCD.
constexpr int WG_XCD_CHUNKS = 64;

// A tile's sums for one site chunk.  Several chunks: split-K partials stored
// as the MFMA result fragments, the layout the reduce reads: per chunk,
// 16 x 16 blocks (bm, bn) for bm < ceil(m_rows / 16), bn < ceil(c_out / 16)
// (blocks past the rows and columns read back are not stored), block
// bm * NB + bn holding 64 lanes x 4 floats, lane 16 g + c the rows 4 g .. 4 g + 3
// of column c; one 16-byte store per lane and block.  A single chunk: the sums
// are final and go to dW / db.
template <class C>
__device__ inline void store_wgrad_tile(const WGradArgs& a, const f32x4 (&acc)[C::TM][C::TN], int chunk, int nch,
                                        int m0, int n0, int wm, int wn, int lane, int m_rows, int m_gather) {
  const int g = lane >> 4, c16 = lane & 15;
  if (nch > 1) {
    const int MB = (m_rows + 15) / 16, NB = (a.c_out + 15) / 16;
    float* part = a.part + (int64_t)chunk * MB * NB * 256;
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int j = 0; j < C::TN; ++j) {
        const int bm = (m0 + C::row(wm, i)) / 16, bn = (n0 + C::col(wn, j)) / 16;
        if (bm < MB && bn < NB) *(f32x4*)(part + ((int64_t)(bm * NB + bn) * 64 + lane) * 4) = acc[i][j];
      }
    return;
  }
  // a lane's 4 rows 4 g .. 4 g + 3 of block i share one window position f
  // (cseg and the rows' first index are multiples of 4): one division per block
  const float rcp_cseg = 1.f / (float)a.cseg;
#pragma unroll
  for (int i = 0; i < C::TM; ++i) {
    const int mb = m0 + C::row(wm, i) + g * 4;
    const int f = div_small(mb, a.cseg, rcp_cseg), c = mb - f * a.cseg;
    int idx[4];
    bool wr[4], br[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      wr[r] = mb + r < m_gather && c + r < a.c_in;
      br[r] = mb + r == a.m_ones && a.db;
      idx[r] = (f * a.c_in + c + r) * a.c_out;
    }
#pragma unroll
    for (int j = 0; j < C::TN; ++j) {
      const int nn = n0 + C::col(wn, j) + c16;
      if (nn >= a.c_out) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (wr[r])
          a.dW[idx[r] + nn] = acc[i][j][r];
        else if (br[r])
          a.db[nn] = acc[i][j][r];
      }
    }
  }
}

// Pair swizzle of an LDS row of sites for the transpose reads below: the
// 32-byte pair p of row r sits at pair slot p ^ swz(r).  A wavefront's read
// touches rows {0..3, 8..11} (+ 16, + 4, + 32) in each half, so the swizzle
// spreads each such set of eight rows over all 64 banks: 256-byte rows by
// (r % 4, r / 8 % 2), 128-byte rows (two per bank sweep) by (r / 2 % 2, r / 8 % 2).
template <int ROW_BYTES>
__device__ inline int site_row_swz(int r) {
  static_assert(ROW_BYTES == 256 || ROW_BYTES == 128, "row width");
  if constexpr (ROW_BYTES == 256)
    return (r & 3) | (((r >> 3) & 1) << 2);
  else
    return ((r >> 1) & 1) | (((r >> 3) & 1) << 1);
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// 8 consecutive sites of one column as an MFMA operand (k = sites): two LDS
// transpose reads of 4 sites each.  Within each 16-lane group, lane q reads
// 4 columns (4 (q % 4) .. + 3) of site row q / 4 and receives column q of the
// group's 4 rows; `p` points at lane q's 4 columns of the group's first row.
template <int ROW>
__device__ inline bf16x8 tr_operand(const __bf16* p) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)lds_addr(p));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)lds_addr(p + 4 * ROW));
  const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

// acc += G_slab^T * delta_slab for one slab of BKS sites held as [site][column]
// (A: BM columns, B: BN columns, pair-swizzled rows).  ONES: this wave's rows
// hold the bias row m_loc, whose operand is 1 for each of the slab's first
// `valid` sites and 0 after.
template <class C, int BKS, bool ONES>
__device__ inline void mma_slab_tr(const __bf16* As, const __bf16* Bs, f32x4 (&acc)[C::TM][C::TN], int wm, int wn,
                                   int lane, int m_loc, int valid) {
  constexpr int BM = C::BM, BN = C::BN;
  const int g = lane >> 4, q = lane & 15;
  const int e4 = 4 * (q & 3);
#pragma unroll
  for (int kb = 0; kb < BKS; kb += C::KB) {
    const int row = kb + 8 * g + (q >> 2);
    const int ha = site_row_swz<BM * 2>(row), hb = site_row_swz<BN * 2>(row);
    bf16x8 bv[C::TN];
#pragma unroll
    for (int j = 0; j < C::TN; ++j) bv[j] = tr_operand<BN>(Bs + row * BN + (((C::col(wn, j) / 16) ^ hb) << 4) + e4);
#pragma unroll
    for (int i = 0; i < C::TM; ++i) {
      bf16x8 av = tr_operand<BM>(As + row * BM + (((C::row(wm, i) / 16) ^ ha) << 4) + e4);
      if constexpr (ONES) {
        if (C::row(wm, i) + q == m_loc) {
#pragma unroll
          for (int e = 0; e < 8; ++e) av[e] = (__bf16)(kb + 8 * g + e < valid ? 1.f : 0.f);
        }
      }
#pragma unroll
      for (int j = 0; j < C::TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv[j], acc[i][j], 0, 0, 0);
    }
  }
}

// The same for float32, whose 16x16x4 MFMA takes one site per lane group: lane
// (g, q) reads column q of a 16-column block at site kb + g, straight from the
// slab as stored.  Blocks are swizzled by the site (block b of site r at block
// slot b ^ (r % 4)), so the four sites of a read lie in different banks.  Only
// the wave's first LM row blocks and LN column blocks are computed.
template <class C, int BKS, bool ONES, int LM, int LN>
__device__ inline void mma_slab_sites(const float* As, const float* Bs, f32x4 (&acc)[C::TM][C::TN], int wm, int wn,
                                      int lane, int m_loc, int valid) {
  constexpr int BM = C::BM, BN = C::BN;
  const int g = lane >> 4, q = lane & 15;
#pragma unroll
  for (int kb = 0; kb < BKS; kb += 4) {
    const int site = kb + g;
    float av[LM], bv[LN];
#pragma unroll
    for (int i = 0; i < LM; ++i) {
      av[i] = As[site * BM + (((C::row(wm, i) / 16) ^ g) << 4) + q];
      if constexpr (ONES)
        if (C::row(wm, i) + q == m_loc) av[i] = site < valid ? 1.f : 0.f;
    }
#pragma unroll
    for (int j = 0; j < LN; ++j) bv[j] = Bs[site * BN + (((C::col(wn, j) / 16) ^ g) << 4) + q];
#pragma unroll
    for (int i = 0; i < LM; ++i)
#pragma unroll
      for (int j = 0; j < LN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
  }
}

// s_waitcnt vmcnt(BASE + STEP x steps) lgkmcnt(0), steps a run-time value in 0 .. 3
template <int BASE, int STEP>
__device__ inline void wait_vmcnt_steps(int steps) {
  switch (steps) {
    case 0: wait_vmcnt<BASE>(); break;
    case 1: wait_vmcnt<BASE + STEP>(); break;
    case 2: wait_vmcnt<BASE + 2 * STEP>(); break;
    default: wait_vmcnt<BASE + 3 * STEP>(); break;
  }
}

// Weight-gradient GEMM, split over sites (the K dimension).  One launch serves a
// group of layers: workgroup tile t belongs to the layer l with tile_beg[l] <= t
// < tile_beg[l + 1].  The operand slabs (BKS sites) go from memory straight into
// LDS as stored, one site per LDS row (bf16: buffer loads with an LDS
// destination, an offset past the buffer reads zero; float32: loads from 64-bit
// addresses), and the MFMA operands are read across sites (bf16: with the LDS
// transpose read).  NST stages: the loads of NST - 1 slabs fly while one is
// multiplied, one barrier per slab.  The window rows of a slab reach LDS the
// same way, into a ring of NST slots, issued with the operand loads NST - 1
// slabs before the ones that read them (so that waiting for a slab's operands
// also covers the window rows of the slab NST - 1 after it).  Every wave issues
// the same number of window-row loads per slab (unused ones read zero into a
// spare row), which keeps the wait counts compile-time constants.
template <typename T, class C, int BKS, int NST>
__global__ void __launch_bounds__(C::NT) k_wgrad(WGradGroup grp, ExtraTask x) {
  constexpr bool B16 = sizeof(T) == 2;
  constexpr int VE = C::VE;
  constexpr int BM = C::BM, BN = C::BN, NT = C::NT, BK = C::BK;
  static_assert(NT == 256 && BM == 128 && BK % BKS == 0 && BKS % (B16 ? C::KB : 4) == 0 && NST >= 2 && NST <= 4,
                "slab and thread layout below");
  constexpr int ACH = BM / VE, BCH = BN / VE;  // 16-byte chunks per LDS row
  constexpr int AV = BKS * ACH / NT, BV = BKS * BCH / NT;
  static_assert(AV * NT == BKS * ACH && BV * NT == BKS * BCH, "slab splits evenly over the threads");
  constexpr int LPS = AV + BV;                       // operand loads per thread and slab
  constexpr int STG = BKS * (BM + BN);               // elements per stage
  // window-row entries per slab, rounded up to whole 64-dword loads: a load's
  // lanes past the slab's entries still write (zeros) to LDS
  constexpr int RSLOT = (BKS * AMAX + 63) / 64 * 64;
  constexpr int NRW = (RSLOT / 64 + 3) / 4;          // window-row loads per wave and slab
  __shared__ __attribute__((aligned(16))) T smem[NST * STG];
  __shared__ __attribute__((aligned(16))) int32_t Rr[NST * RSLOT + 64];  // + a spare row for unused loads

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / C::WN, wn = wave % C::WN;
  if (run_extra<T>(x)) return;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const uint32_t lds_s = lds_addr(smem), lds_r = lds_addr(Rr), lds_spare = lds_r + NST * RSLOT * 4;
  // this thread's 16-byte LDS slots, the same in every slab: A rows tid / ACH +
  // j NT / ACH at slot tid % ACH, B rows tid / BCH + j NT / BCH at slot tid % BCH
  // (the row bits the swizzle reads do not change with j), and the logical
  // column chunk each slot holds
  const int ra0 = tid / ACH, ta = tid % ACH, rb0 = tid / BCH, tb = tid % BCH;
  static_assert(NT / ACH % (B16 ? 16 : 4) == 0 && NT / BCH % (B16 ? 16 : 4) == 0, "the row bits the swizzle reads");
  int ca, cb;
  if constexpr (B16) {
    ca = 2 * ((ta >> 1) ^ site_row_swz<BM * 2>(ra0)) + (ta & 1);
    cb = 2 * ((tb >> 1) ^ site_row_swz<BN * 2>(rb0)) + (tb & 1);
  } else {
    ca = 4 * ((ta >> 2) ^ (ra0 & 3)) + (ta & 3);
    cb = 4 * ((tb >> 2) ^ (rb0 & 3)) + (tb & 3);
  }

  for (int t = blockIdx.x; t < grp.tile_beg[grp.n]; t += own_grid(x)) {
    int l = 0;
    while (l + 1 < grp.n && t >= grp.tile_beg[l + 1]) ++l;
    const WGradArgs& a = grp.L[l];
    const int tile = t - grp.tile_beg[l];
    const int rows = a.rows_dev ? *a.rows_dev + a.rows_add : a.rows_host;
    const int tiles_m = a.Mpad / BM, tiles_n = a.Npad / BN;
    const int nch = wgrad_chunks(a);
    const int per = ((rows + nch - 1) / nch + BK - 1) / BK * BK;
    const int m_gather = a.A * a.cseg;
    const int m_rows = a.m_ones >= 0 ? a.m_ones + 1 : m_gather;  // rows of dW / db that are read back
    // Many chunks: all tiles of a chunk on one XCD (workgroups are dealt
    // round-robin to the eight), chunk c on XCD c % 8, so that its sites' rows,
    // which every tile of the chunk reads, come through one L2.  Few chunks would
    // leave XCDs idle.
    const int tpc = tiles_m * tiles_n;
    int chunk = tile / tpc, ct = tile - chunk * tpc;
    if (nch >= WG_XCD_CHUNKS) {
      const int i = tile >> 3;
      chunk = i / tpc * 8 + (tile & 7);
      ct = i - i / tpc * tpc;
    }
    if (chunk >= nch) continue;  // fewer rows than the plan allowed for
    const int tm = ct / tiles_n, tn = ct - tm * tiles_n;
    const int m0 = tm * BM, n0 = tn * BN;
    const int o_beg = chunk * per;
    const int o_end = min(rows, o_beg + per);
    const int nsl = o_end > o_beg ? (o_end - o_beg + BKS - 1) / BKS : 0;
    f32x4 acc[C::TM][C::TN];
#pragma unroll
    for (int i = 0; i < C::TM; ++i)
#pragma unroll
      for (int j = 0; j < C::TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    const int A = a.A;
    const int ma = m0 + VE * ca;  // first column of this thread's A chunk: window position fa, channel cola
    const bool a_col = ma < m_gather;
    const int fa = a_col ? ma / a.cseg : 0;
    const int cola = ma - fa * a.cseg;
    const int nb = n0 + VE * cb;
    const bool b_col = nb < a.dsrc_cols;
    const bool has_r = a.rmap != nullptr;
    const int r_loads = has_r ? (BKS * A + 63) / 64 : 0;  // 64-dword loads that carry window rows
    // (held in registers: the loop's compiler fences would otherwise reload
    // them from the kernel arguments on every slab)
    const int src_stride = a.src_stride, dsrc_stride = a.dsrc_stride;
    const u32x4 rsA = buffer_rsrc(a.src, GATHER_SRC_BYTES);
    const u32x4 rsB = buffer_rsrc(a.dsrc, GATHER_SRC_BYTES);
    const u32x4 rsR = buffer_rsrc(a.rmap, GATHER_SRC_BYTES);
    const T* src = (const T*)a.src;
    const T* dsrc = (const T*)a.dsrc;
    const uint32_t src_bytes = (uint32_t)src_stride * (uint32_t)sizeof(T), dsrc_bytes = (uint32_t)dsrc_stride * (uint32_t)sizeof(T);
    const int32_t* rmap = a.rmap;
    const void* zero = a.zero;
    // this wave's blocks that hold part of the result
    const int live_m = __builtin_amdgcn_readfirstlane(
        (min(m_rows - m0, BM) - wm * 16 + 16 * C::WM - 1) / (16 * C::WM));
    const int live_n = __builtin_amdgcn_readfirstlane(
        (min(a.c_out - n0, BN) - wn * 16 + 16 * C::WN - 1) / (16 * C::WN));
    // window rows of slab s (sites ob .. ob + BKS - 1, A entries each,
    // contiguous) into ring slot s % NST: wave w's i-th load takes dwords
    // 64 k .. 64 k + 63, k = w + 4 i; NRW loads per wave whatever A and s
    auto issue_rows = [&](int s) {
      const int ob = o_beg + s * BKS;
      const uint32_t dst = lds_r + (uint32_t)((s % NST) * RSLOT) * 4u;
#pragma unroll
      for (int i = 0; i < NRW; ++i) {
        const int k = wave_u + 4 * i;
        const bool used = s < nsl && k < r_loads;
        const int d = 64 * k + lane;
        const bool live = used && d < BKS * A && ob * A + d < o_end * A;
        const uint32_t to = used ? dst + (uint32_t)k * 256u : lds_spare;
        if constexpr (B16)
          dma4(rsR, to, live ? (uint32_t)(ob * A + d) * 4u : GATHER_SRC_BYTES);
        else
          dma4_at(to, (const void*)(live ? (uint64_t)(rmap + ((int64_t)ob * A + d)) : (uint64_t)zero));
      }
    };
    // operand slab s into stage s % NST, reading its window rows from ring slot s % NST
    auto issue_slab = [&](int s) {
      const int ob = o_beg + s * BKS;
      const uint32_t sa = lds_s + (uint32_t)((s % NST) * STG * (int)sizeof(T)), sb = sa + BM * BKS * (int)sizeof(T);
      const int32_t* R = Rr + (s % NST) * RSLOT;
      int srow[AV];
#pragma unroll
      for (int j = 0; j < AV; ++j) {  // every window row read before the first load goes out
        const int r = ra0 + j * (NT / ACH);
        const int o = ob + r;
        srow[j] = has_r ? R[r * A + fa] : o;
        if (!a_col || o >= o_end) srow[j] = -1;
      }
#pragma unroll
      for (int j = 0; j < AV; ++j) {
        const uint32_t to = sa + (uint32_t)(wave_u * 64 + j * NT) * 16u;
        if constexpr (B16)
          dma16(rsA, to, srow[j] >= 0 ? (uint32_t)(srow[j] * src_stride + cola) * 2u : GATHER_SRC_BYTES);
        else
          dma16_at(to, (const void*)(srow[j] >= 0 ? (uint64_t)(src + cola) + (uint64_t)(uint32_t)srow[j] * src_bytes
                                                  : (uint64_t)zero));
      }
#pragma unroll
      for (int j = 0; j < BV; ++j) {
        const int o = ob + rb0 + j * (NT / BCH);
        const uint32_t to = sb + (uint32_t)(wave_u * 64 + j * NT) * 16u;
        const bool on = b_col && o < o_end;
        if constexpr (B16)
          dma16(rsB, to, on ? (uint32_t)(o * dsrc_stride + nb) * 2u : GATHER_SRC_BYTES);
        else
          dma16_at(to, (const void*)(on ? (uint64_t)(dsrc + nb) + (uint64_t)(uint32_t)o * dsrc_bytes : (uint64_t)zero));
      }
    };
    // the bias row (softmax layer): the wave whose rows hold it patches its operand
    const int m_loc = a.m_ones - m0;
    const bool ones = a.m_ones >= 0 && m_loc >= 0 && m_loc < BM && m_loc / 16 % C::WM == wm;

    if (nsl > 0) {
      // window rows of the first NST - 1 slabs, their operands, then (once
      // every wave has read those ring slots) the window rows of the next NST - 1
      for (int p = 0; p < NST - 1; ++p) issue_rows(p);
      asm volatile("" ::: "memory");
      wait_vmcnt<0>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      for (int p = 0; p < NST - 1; ++p)
        if (p < nsl) issue_slab(p);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0) only: the operand loads stay in flight
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      for (int p = NST - 1; p < 2 * NST - 2; ++p) issue_rows(p);
    }
    // the slab loop, with the bias-row patch compiled into a copy of its own
    // (a branch per slab made the compiler copy the accumulators between the
    // two MFMA sequences on every slab)
    auto slab_loop = [&](auto ones_c, auto lm_c, auto ln_c) {
      constexpr bool ONES = decltype(ones_c)::value;
      constexpr int LM = decltype(lm_c)::value, LN = decltype(ln_c)::value;
      for (int s = 0; s < nsl; ++s) {
        // slab s and the window rows of slab s + NST - 1 have landed (this
        // wave's, and after the barrier every wave's); every wave is done with
        // slab s - 1 and with the ring slot refilled below.  Loads issued after
        // those may stay in flight: the window rows issued since (NRW per slab)
        // and the operand slabs after s that exist.
        asm volatile("" ::: "memory");
        if constexpr (NST == 2) {
          wait_vmcnt<0>();
        } else {
          // issued after the last load slab s needs (its operands, or at s <=
          // NST - 2 the prologue's window rows of slab s + NST - 1): NST - 2
          // batches of window rows, and the operand slabs i + NST - 1 < nsl
          // issued by iterations i = max(0, s - NST + 2) .. s - 1
          const int lo = max(0, s - NST + 2), hi = min(s - 1, nsl - NST);
          wait_vmcnt_steps<(NST - 2) * NRW, LPS>(hi >= lo ? hi - lo + 1 : 0);
        }
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        issue_rows(s + 2 * NST - 2);
        if (s + NST - 1 < nsl) issue_slab(s + NST - 1);
        const T* As = smem + (s % NST) * STG;
        const int valid = o_end - (o_beg + s * BKS);
        if constexpr (B16)
          mma_slab_tr<C, BKS, ONES>(As, As + BM * BKS, acc, wm, wn, lane, m_loc, valid);
        else
          mma_slab_sites<C, BKS, ONES, LM, LN>(As, As + BM * BKS, acc, wm, wn, lane, m_loc, valid);
      }
    };
    // (float32 also by the live blocks of this wave, as in the gather GEMM; every
    // wave passes the same barriers in whichever copy it runs)
    constexpr std::integral_constant<int, C::TM> all_m{};
    constexpr std::integral_constant<int, C::TN> all_n{};
    if (ones)
      slab_loop(std::integral_constant<bool, true>{}, all_m, all_n);
    else if constexpr (B16)
      slab_loop(std::integral_constant<bool, false>{}, all_m, all_n);
    else
      with_count<C::TM == 4 ? 2 : 1, C::TM>(live_m, [&](auto lm_c) {
        with_count<2, C::TN>(live_n, [&](auto ln_c) { slab_loop(std::integral_constant<bool, false>{}, lm_c, ln_c); });
      });

    store_wgrad_tile<C>(a, acc, chunk, nch, m0, n0, wm, wn, lane, m_rows, m_gather);
  }
}

// dW (and db) from the split-K partials, for a group of layers (block b
// belongs to layer l with blk_beg[l] <= b < blk_beg[l + 1]).  A block has G
// thread groups (G = 16, or fewer when there are fewer chunks) of 256/G
// threads, one 16-byte fragment quad of the partial layout (rows 4 g .. 4 g + 3
// of one column) per thread of a group; group g sums chunks g, g+G, ...; the G
// group sums are added in a fixed order.
__global__ void __launch_bounds__(256) k_wgrad_reduce(WGradGroup grp) {
  __shared__ f32x4 red[256];
  int l = 0;
  while (l + 1 < grp.n && (int)blockIdx.x >= grp.blk_beg[l + 1]) ++l;
  const WGradArgs& a = grp.L[l];
  const int nch = wgrad_chunks(a);
  if (nch <= 1) return;  // the weight-gradient kernel wrote the results
  const int G = grp.G[l];
  const int E = 256 / G;  // quads per block
  const int m_gather = a.A * a.cseg;
  const int m_rows = a.m_ones >= 0 ? a.m_ones + 1 : m_gather;
  const int MB = (m_rows + 15) / 16, NB = (a.c_out + 15) / 16;
  const int64_t total = (int64_t)MB * NB * 64;
  const int el = threadIdx.x % E, grpi = threadIdx.x / E;
  const int64_t t = (int64_t)((int)blockIdx.x - grp.blk_beg[l]) * E + el;
  f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
  if (t < total) {
    const float* part = a.part + t * 4;
    const int64_t cstride = total * 4;
    for (int ch = grpi; ch < nch; ch += G) s += *(const f32x4*)(part + ch * cstride);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  if (grpi != 0 || t >= total) return;
  s = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int g = 0; g < G; ++g) s += red[g * E + el];
  const int blk = (int)(t >> 6), ln = (int)(t & 63);
  const int bm = blk / NB, bn = blk - bm * NB;
  const int n = 16 * bn + (ln & 15);
  if (n >= a.c_out) return;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = 16 * bm + 4 * (ln >> 4) + r;
    if (m < m_gather) {
      const int f = m / a.cseg, c = m - f * a.cseg;
      if (c < a.c_in) a.dW[((int64_t)f * a.c_in + c) * a.c_out + n] = s[r];
    } else if (m == a.m_ones) {
      if (a.db) a.db[n] = s[r];
    }
  }
}

template <typename T>
__global__ void __launch_bounds__(256) k_row0_dx(Row0Args r) {
  row0_dx_block<T>(r, blockIdx.x);
}

static int device_grid_limit() { return 256 * 8; }

template <typename T, class C>
static void launch_cfg(const GemmArgs& a, int64_t max_rows, hipStream_t st) {
  const int64_t span = max_rows - a.row_begin;
  const int64_t tiles = ((span + C::BM - 1) / C::BM) * (a.Npad / C::BN) * a.ksplit;
  const int grid = deal_grid(tiles, device_grid_limit(), deal_by_xcd(a.Npad / C::BN, a.rmap != nullptr, a.A, a.ksplit)) +
                   (a.x.kind ? a.x.blocks : 0);
  const bool timed = a.t_start || a.t_stop;
  // the pooling-backward epilogue and the masked store have instantiations of
  // their own (their extra loads and sums would otherwise cost every launch
  // registers)
  const int mode = gemm_mode(a.pool_fwd, a.epi == EPI_STORE_MASK, a.route, a.route_ac, a.ksplit);
  void (*kern)(GemmArgs) = mode == POOL_FWD_MODE ? k_gemm_gather<T, C, POOL_FWD_MODE>
                           : mode == MASK_MODE   ? k_gemm_gather<T, C, MASK_MODE>
                           : mode == PLAIN_MODE  ? k_gemm_gather<T, C, PLAIN_MODE>
                           : mode == 4           ? k_gemm_gather<T, C, 4>
                                                 : k_gemm_gather<T, C, 0>;
  // the window table and the chunk words: a workgroup's LDS follows A and K
  const size_t lds = ((size_t)C::BM * a.A + (sizeof(T) == 2 && a.A > 1 ? a.Kpad / C::VE : 0)) * sizeof(int32_t);
  if (timed)
    hipExtLaunchKernelGGL(kern, dim3(grid), dim3(C::NT), lds, st, a.t_start,
                          a.ksplit > 1 && !a.partials_only ? nullptr : a.t_stop, 0, a);
  else
    hipLaunchKernelGGL(kern, dim3(grid), dim3(C::NT), lds, st, a);
  if (a.ksplit > 1 && !a.partials_only) {
    const int64_t total = span * ((a.out_cols + 3) / 4);
    const int g2 = (int)std::min<int64_t>(std::max<int64_t>((total + 255) / 256, 1), 4096);
    if (timed)
      hipExtLaunchKernelGGL(k_gemm_splitk_reduce<T>, dim3(g2), dim3(256), 0, st, nullptr, a.t_stop, 0, a);
    else
      hipLaunchKernelGGL(k_gemm_splitk_reduce<T>, dim3(g2), dim3(256), 0, st, a);
  }
}

template <typename T>
static void launch_gemm_t(const GemmArgs& a, int64_t max_rows, hipStream_t st) {
  switch (a.cfg) {
    case 0: launch_cfg<T, C128x128<T>>(a, max_rows, st); break;
    case 1: launch_cfg<T, C128x64<T>>(a, max_rows, st); break;
    case 2: launch_cfg<T, C64x64<T>>(a, max_rows, st); break;
    default: launch_cfg<T, C32x64<T>>(a, max_rows, st); break;
  }
}

hipError_t launch_gemm(bool bf16, const GemmArgs& args, int64_t max_rows, hipStream_t st) {
  if (max_rows - args.row_begin <= 0) return hipSuccess;
  if (max_rows > INT32_MAX) return hipErrorInvalidValue;
  if (args.A < 1 || args.A > AMAX) return hipErrorInvalidValue;  // window tables hold at most AMAX entries a row
  GemmArgs a = args;
  a.rows_cap = (int32_t)max_rows;
  if (a.pool_fwd && (a.route || a.ksplit != 1 || a.row_begin != 0 || !a.pslot ||
                     !a.pool_out || !a.pool_argmax || !a.rows_dev ||
                     (a.epi != EPI_BIAS_RELU && a.epi != EPI_BIAS_LRELU)))
    return hipErrorInvalidValue;
  if (a.epi == EPI_STORE_MASK && a.bias) return hipErrorInvalidValue;
  if (a.sums && (a.epi != EPI_STORE_MASK || a.ksplit != 1 || a.row_begin != 1 || !a.pr.part || a.pr.cp != a.out_cols ||
                 (max_rows - a.row_begin + gemm_bm(bf16, a.cfg) - 1) / gemm_bm(bf16, a.cfg) > a.pr.PM))
    return hipErrorInvalidValue;
  if (a.route) {  // pooling backward in the epilogue: one partial per row tile
    const int bm = gemm_bm(bf16, a.cfg);
    if (a.epi != EPI_STORE || a.bias || a.ksplit != 1 || (a.route_ac != 0 && a.route_ac != 4) ||
        !a.pr.part || !a.pr.Rp || !a.pr.argmax || !a.pr.dZ || !a.pr.X_pool || (a.route_ac == 4 && !a.pr.gmask) ||
        a.pr.cp != a.out_cols || a.pr.stride != a.pr.cp || (max_rows - a.row_begin + bm - 1) / bm > a.pr.PM)
      return hipErrorInvalidValue;
  }
  if (a.cfg == GEMM_DIRECT) return launch_gemm_direct(bf16, a, max_rows, st);
  if (bf16)
    launch_gemm_t<__bf16>(a, max_rows, st);
  else
    launch_gemm_t<float>(a, max_rows, st);
  return hipGetLastError();
}

GemmPlan plan_gemm(bool bf16, int64_t max_rows, int N, int K, GemmKind kind) {
  const bool short_rows = kind == GEMM_ROUTED;
  // Launches with few output tiles (at the row bound) go to the
  // direct-operand kernel, whose waves split K and so keep many loads in flight
  // per tile; launches with more tiles keep the LDS-tiled kernel, whose slabs
  // stream through LDS stages shared by the tile's waves.  (Measured on the
  // pen-stroke DeepCNet(5,50), bf16, batch 100, tiles counted as 32 x 64 at the
  // row bound: forward with the pooling forward, 204 tiles, 10.0 us direct against
  // 12.0 LDS-tiled; the softmax layer's forward, 236 tiles, 7.2 us direct against
  // 6.6 LDS-tiled.  Input gradients with the pooling backward, K 1200 at 52 tiles
  // 12.5 us direct against 7.6 with a split-K reduce and a pooling pass (4.5 + 7.5)
  // behind it, K 1000 at 364 tiles 18.9 against 16.1, but K 160 at 420 tiles 8.5
  // against 9.4: up to 256 tiles, or 600 for K <= 320.  The last convolution's
  // forward, 20 tiles of K 1000, 10.2 us direct against 5.7 with a reduce of 4.6;
  // 50 tiles of K 2000 15.1 against 8.0 and 4.6: split K above 1024.)
  // float32 (one lane holds 4 k, not 8: twice the loads per k block and sixteen
  // times the MFMA time) goes there for up to 128 tiles and K <= 512, where it
  // saves the split-K reduce and lets the pooling passes ride in the epilogue:
  // DeepCNet(4,20) at batch 8, K = 80 .. 320: forwards 6.2 + 3.5 (reduce) + 2.5
  // (pooling) -> 7.5 us, input gradients 7.0 + 3.7 + 4.8 -> 13.7 us; but K = 1000
  // at 20 tiles 20.1 us against 6.7 + 5.0.
  // (Each of these limits lies between the one or two launches named on either side
  // of it; where exactly, between them, was not measured.)
  const int64_t direct_tiles = ((max_rows + DIRECT_BM - 1) / DIRECT_BM) * ((N + DIRECT_BN - 1) / DIRECT_BN);
  const int64_t most = !bf16 ? 128 : kind == GEMM_ROUTED ? (K <= 320 ? 600 : 256) : kind == GEMM_POOLED ? 256 : 128;
  if (direct_tiles <= most && K <= (!bf16 ? 512 : kind == GEMM_PLAIN ? 1024 : 2048)) {
    GemmPlan p;
    p.cfg = GEMM_DIRECT;
    p.BN = DIRECT_BN;
    p.Npad = (int)round_up(N, DIRECT_BN);
    p.Kpad = (int)round_up(K, 64);
    p.ksplit = 1;
    return p;
  }
  // Tile width: 128 when that pads N no more than 64 does and still gives >= 256
  // tiles; otherwise 64-wide tiles with the tallest of 128/64/32 rows that gives
  // >= 256 tiles.  K is split when even 32-row tiles leave the GPU mostly idle.
  // short_rows (an epilogue that routes every row through its pooling window,
  // a thread's rows one after another): at most 64 rows per tile, so that each
  // thread routes two rows, not four or eight (measured on the pen-stroke
  // DeepCNet(5,50) input gradient of the second level: 31.9 -> 25.8 us).
  const int BK = bf16 ? 64 : 32;
  const int64_t n128 = (N + 127) / 128 * 128, n64 = (N + 63) / 64 * 64;
  auto tiles = [&](int bm, int64_t npad, int bn) { return ((max_rows + bm - 1) / bm) * (npad / bn); };
  GemmPlan p;
  // float32, whose MFMAs take sixteen times as long: smaller tiles while a launch
  // has few of them (a compute unit with one tile more than the others holds the
  // launch up for its whole time: DeepCNet(5,50)'s fourth forward 50.4 us in 264
  // 128 x 64 tiles, 41.6 in 528 of 64 x 64; its third input gradient 31.7 us in
  // 770 64 x 64 tiles at the row bound, 28.5 in 32 x 64), and 128 rows only where K
  // is long enough to make up for a taller tile's setup and epilogue (40 channels
  // wide, K = 120: 14.3 us against 12.4 with 64 rows; 150 wide, K = 400: 40.0
  // against 45.1).
  if (!bf16) {
    const bool tall = !short_rows && K > 4 * BK;
    p.cfg = tall && n128 <= n64 && tiles(128, n128, 128) >= 256 ? 0
            : tall && tiles(128, n64, 64) >= 512                ? 1
            : tiles(64, n64, 64) >= 1024                        ? 2
                                                                : 3;
  } else if (!short_rows && n128 <= n64 && tiles(128, n128, 128) >= 256)
    p.cfg = 0;
  else if (!short_rows && tiles(128, n64, 64) >= 256)
    p.cfg = 1;
  else if (tiles(64, n64, 64) >= 256)
    p.cfg = 2;
  else
    p.cfg = 3;
  const GemmTile t = gemm_tile(bf16, p.cfg);
  p.BN = t.BN;
  p.Npad = (int)round_up(N, t.BN);
  p.Kpad = (int)round_up(K, BK);
  const int64_t tl = tiles(t.BM, p.Npad, t.BN);
  const int kslabs = p.Kpad / BK;
  p.ksplit = 1;
  if (tl < 128 && kslabs >= 4) p.ksplit = (int)std::max<int64_t>(1, std::min<int64_t>(kslabs / 2, (256 + tl - 1) / tl));
  return p;
}

hipError_t launch_wgrad(bool bf16, int cfg, const WGradArgs* layers, int n, hipStream_t st, const ExtraTask* extra) {
  // cfg: 0 = 128 x 128 tiles, 1 = 128 x 64
  if (n < 1 || n > MAX_WG_LAYERS) return hipErrorInvalidValue;
  const ExtraTask x = extra ? *extra : ExtraTask{};
  if (x.kind && (x.blocks < 1 || (x.kind != 1 && x.kind != 3))) return hipErrorInvalidValue;
  const int BN = cfg == 0 ? 128 : 64;
  WGradGroup g{};
  g.n = n;
  g.tile_beg[0] = 0;
  for (int l = 0; l < n; ++l) {
    if (layers[l].A < 1 || layers[l].A > AMAX || (layers[l].nchunks > 1 && !layers[l].nch_dev))
      return hipErrorInvalidValue;
    g.L[l] = layers[l];
    const int nch = layers[l].nchunks;  // whole groups of eight where chunks may be dealt by XCD
    g.tile_beg[l + 1] = g.tile_beg[l] + (layers[l].Mpad / 128) * (layers[l].Npad / BN) *
                                            (nch >= WG_XCD_CHUNKS ? (nch + 7) / 8 * 8 : nch);
  }
  const int grid = std::min(std::max(g.tile_beg[n], 1), device_grid_limit()) + (x.kind ? x.blocks : 0);
  // sites per slab and LDS stages: as many stages as leave two (128 x 128) or
  // three (128 x 64) workgroups per compute unit
  if (bf16) {
    if (cfg == 0)
      hipLaunchKernelGGL((k_wgrad<__bf16, C128x128<__bf16>, 32, 4>), dim3(grid), dim3(256), 0, st, g, x);
    else
      hipLaunchKernelGGL((k_wgrad<__bf16, C128x64<__bf16>, 32, 3>), dim3(grid), dim3(256), 0, st, g, x);
  } else {
    if (cfg == 0)
      hipLaunchKernelGGL((k_wgrad<float, GCfg<float, 2, 2, 4, 4>, 16, 4>), dim3(grid), dim3(256), 0, st, g, x);
    else
      hipLaunchKernelGGL((k_wgrad<float, C128x64<float>, 16, 4>), dim3(grid), dim3(256), 0, st, g, x);
  }
  return hipGetLastError();
}

hipError_t launch_wgrad_reduce(const WGradArgs* layers, int n, hipStream_t st) {
  WGradGroup g{};
  g.blk_beg[0] = 0;
  for (int l = 0; l < n; ++l) {
    const WGradArgs& a = layers[l];
    if (a.nchunks <= 1) continue;  // the weight-gradient kernel wrote the results
    const int m_rows = a.m_ones >= 0 ? a.m_ones + 1 : a.A * a.cseg;
    // fragment quads of the partial layout: 16 x 16 blocks over the rows and
    // columns read back, 64 per block
    const int64_t total = (int64_t)((m_rows + 15) / 16) * ((a.c_out + 15) / 16) * 64;
    const int G = a.nchunks >= 16 ? 16 : (a.nchunks >= 8 ? 8 : (a.nchunks >= 4 ? 4 : 2));
    const int E = 256 / G;
    g.L[g.n] = a;
    g.G[g.n] = G;
    g.blk_beg[g.n + 1] = g.blk_beg[g.n] + (int)((total + E - 1) / E);
    ++g.n;
  }
  if (g.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_wgrad_reduce, dim3(g.blk_beg[g.n]), dim3(256), 0, st, g);
  return hipGetLastError();
}

hipError_t launch_row0_dx(bool bf16, const void* W, const float* D0, int32_t A, int32_t c_in, int32_t c_out,
                          int32_t cp_in, void* grad_in, const void* Y_below, float slope, hipStream_t st) {
  const Row0Args r{W, D0, A, c_in, c_out, cp_in, grad_in, Y_below, slope};
  if (bf16)
    hipLaunchKernelGGL(k_row0_dx<__bf16>, dim3(cp_in), dim3(256), 0, st, r);
  else
    hipLaunchKernelGGL(k_row0_dx<float>, dim3(cp_in), dim3(256), 0, st, r);
  return hipGetLastError();
}

}  // namespace sscn
