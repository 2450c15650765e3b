// symi_expert_fwd / symi_expert_bwd: the expert SwiGLU FFN over replica slots as
// variable-group grouped GEMMs (paper Sec. 2.1; the expert compute of Fig. 5; the
// intra-rank part of the replica gradient reduction of Sec. 4.1 is fused into the
// weight-gradient GEMM, which sums over every row of a class at once).
//
// Six products share one tiled kernel (bf16 inputs, fp32 accumulation on the gfx950
// MFMA 16x16x32 bf16 instruction; fp32 configurations split every value into three bf16 ones or take the fp32 MFMA):
//   FWD1   [u|v] = Xp  * W1^T      + SwiGLU epilogue writing u, v and h = silu(u)*v
//   FWD2   Yp    = H   * W2^T
//   BWD_DH dh    = dYp * W2        turned into du, dv from the saved u, v in the epilogue
//   BWD_DX dXp   = dUV * W1
//   WGRAD2 dW2_e = dYp^T * H       over all rows of class e
//   WGRAD1 dW1_e = dUV^T * Xp      over all rows of class e
// The first four have a variable number of rows per group (one group per slot); a small
// kernel turns slot_offsets into a table of 256-row m-tiles so that no workgroup spans
// two slots.  The last two have a variable reduction length (the rows of a class).  The two
// narrow products (FWD2, BWD_DX) may cut the reduction of their last round's tiles into slices
// that a second small kernel adds up (tail_slices, slice_sum_kernel).
//
// The MFMA is issued with the weight tile as its first operand, so a lane ends up with 4
// consecutive output columns of one output row; the epilogue turns the blocks around through
// LDS so that stores cover whole cache lines.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace symi {

enum { FWD1 = 0, FWD2 = 1, BWD_DH = 2, BWD_DX = 3, WGRAD2 = 4, WGRAD1 = 5, GATE = 6 };   // GATE: symi_router_fwd

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

struct GemmParams {
  const void* A;       // activations (left operand source)
  const void* B;       // weights per slot, or the second activation for weight gradients
  void* C;             // main output
  const void* UV;      // BWD_DH: saved u|v
  void* UVout;         // FWD1: u|v out
  void* H;             // FWD1: h out
  const int32_t* tile_map;      // [4 + 4*i]: header {n_tiles}, then {row0, row1, slot, -}
  const int32_t* tile_map128;   // the 128 x 128 tile's, two words a tile
  const int32_t* slot_offsets;  // weight gradients: class row ranges; small batches: the slots' rows
  int n_slots;
  const int32_t* first_slot;
  long long b_group_stride;     // elements between consecutive slots' weights
  long long c_group_stride;     // elements between consecutive classes' gradients
  int M;   // fixed row count of the output (weight gradients)
  int N;   // output columns (FWD1: f, counted once)
  int K;   // reduction length when fixed
  int d, f;
  const int32_t* class_order;   // weight gradients: classes by decreasing row count
  int per_slot;                 // weight gradients: one output per slot instead of per class
  int skip_empty;               // weight gradients: a group without rows is not written at all
  float* partials;              // partial tiles of sliced reductions (nullptr: never slice)
  int cus;                      // compute units a round of tiles is spread over
};

__device__ __forceinline__ float silu_f(float u) { return u / (1.f + expf(-u)); }
__device__ __forceinline__ float sigmoid_f(float u) { return 1.f / (1.f + expf(-u)); }
// bf16 path: hardware exp2/rcp (relative error ~1e-6, far below the bf16 rounding of the result)
__device__ __forceinline__ float sigmoid_fast(float u) {
  return __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * u));
}

// ---------------------------------------------------------------- m-tile table
// map[0] = number of m-tiles, map[4 + 4i ..] = {first row, end row, slot} of m-tile i (TM = 256 rows), or
// map[4 + 2i ..] = {first row, slot + 2^16 * (rows - 1)} (TM = FEW_BM: the fp32 products, whose workspace holds two words
// for each 64-row tile, and the bf16 small-batch forward products, whose at most 32 rows per slot on average make at most 1.5 S_tot
// tiles, which fit where 256-row tiles would be; TM = MID_BM: the 128 x 128 tile).
// order[c] = the class with the c-th largest number of rows (ties: lower index first).
constexpr int FEW_BM = 64, MID_BM = 128;

// The tables that a call's products read (nullptr: not wanted).  256 and 64 share their place in the workspace: bf16 layers of few rows per slot
// and fp32 layers have no 256-row tiles in a call that has 64-row ones.
struct TileMaps { int32_t *of256, *of128, *of64; };

template <int TM>
__device__ __forceinline__ void write_tile_map(const int32_t* __restrict__ slot_offsets, int S, int32_t* __restrict__ map, int32_t* part) {
  const int tid = threadIdx.x;
  const int per = (S + 255) / 256;
  const int q0 = tid * per, q1 = min(S, q0 + per);
  int mine = 0;
  for (int q = q0; q < q1; ++q) mine += (slot_offsets[q + 1] - slot_offsets[q] + TM - 1) / TM;
  part[tid] = mine;
  __syncthreads();
  for (int o = 1; o < 256; o <<= 1) {  // Hillis-Steele inclusive scan
    const int add = tid >= o ? part[tid - o] : 0;
    __syncthreads();
    part[tid] += add;
    __syncthreads();
  }
  int t = part[tid] - mine;
  if (tid == 255) map[0] = part[255];
  for (int q = q0; q < q1; ++q) {
    const int b = slot_offsets[q], e = slot_offsets[q + 1];
    for (int r = b; r < e; r += TM, ++t) {
      if (TM < GEMM_BM) {
        map[4 + 2 * t + 0] = r;
        map[4 + 2 * t + 1] = q + ((min(e - r, TM) - 1) << 16);
      } else {
        map[4 + 4 * t + 0] = r;
        map[4 + 4 * t + 1] = min(e, r + TM);
        map[4 + 4 * t + 2] = q;
        map[4 + 4 * t + 3] = 0;
      }
    }
  }
  __syncthreads();   // `part` may serve another table
}

__global__ __launch_bounds__(256) void tile_map_kernel(const int32_t* __restrict__ slot_offsets, const int32_t* __restrict__ first_slot, int S,
                                                       int E, TileMaps maps, int32_t* __restrict__ order) {
  __shared__ int32_t part[256];
  __shared__ int32_t rows[1024];
  const int tid = threadIdx.x;
  if (maps.of256) write_tile_map<256>(slot_offsets, S, maps.of256, part);
  if (maps.of128) write_tile_map<MID_BM>(slot_offsets, S, maps.of128, part);
  if (maps.of64) write_tile_map<FEW_BM>(slot_offsets, S, maps.of64, part);
  if (first_slot) {
    for (int e = tid; e < E; e += 256) rows[e] = slot_offsets[first_slot[e + 1]] - slot_offsets[first_slot[e]];
    __syncthreads();
    for (int e = tid; e < E; e += 256) {
      int rank = 0;
      for (int j = 0; j < E; ++j) rank += (rows[j] > rows[e] || (rows[j] == rows[e] && j < e)) ? 1 : 0;
      order[rank] = e;
    }
  }
}

// ---------------------------------------------------------------- bf16 MFMA kernel
// Output tile 256 x 256 per workgroup, reduction step 64, 4 wavefronts in a 2 x 2 grid,
// each owning 128 x 128 outputs = 8 x 8 MFMA 16x16x32 tiles (256 fp32 accumulators per
// lane).  Tiles travel HBM -> LDS with the gfx950 direct-to-LDS loads (16 bytes per
// lane, no staging registers) into two 32 KB stages of the left operand and three of the right
// one, the whole 160 KB of a compute unit.
// With long reductions bound by the matrix pipes at the clock the power limit leaves (c5: busy 67 - 79 % of
// the cycles at 1.6 - 1.74 GHz of 2.4 with random operands; c3, K up to 28672: 68 - 87 %), as long as neither
// loads nor instruction issue leave them idle; with short ones (c2, K = 1024: busy 32 - 64 %) the epilogue,
// which runs with idle pipes, is what is left:
//  - Lead of the loads.  With two stages of both operands the loads of a step had to be issued
//    within two of its four phases and had 2 - 4 phases to land; the third stage of the right operand
//    spreads them evenly over all phases and gives them 2 - 6.
//  - MFMA 16x16x32 instead of 32x32x16: a block sums 32 products before it touches its accumulator,
//    and reads and loads can sit between MFMAs of 16 cycles.  Same bits as 32x32x16.
//  c5's six products 68.7 -> 64.6 (16x16x32) -> 61.3 ms (third stage), c4's 10.17 -> 9.85 -> 9.05, c2's
//  2.73 -> 2.64 -> 2.33; LDS instructions hold 18 - 22 % of the cycles.  Two loads per eight MFMAs instead of
//  one cost 3 %, four 6 %.
// LDS layouts (all conflict-free for the access pattern that reads them):
//   reduction-contiguous operand: [256 rows][64 k], 16-byte chunk c of row r stored at
//     chunk c ^ ((r >> 1) & 7); fragments are plain 16-byte reads.
//   reduction-strided operand (memory [k][r], r contiguous): [64 k][256 r] as loaded,
//     16-byte chunk c of row k stored at c ^ 10*(k & 1) ^ 4*((k >> 1) & 1) ^ 2*((k >> 3) & 1): the
//     32 lanes the LDS serves per cycle (k-rows 0..3 and 8..11, 32 B each) then fall into 64 distinct banks;
//     fragments come from the transposing LDS read (ds_read_b64_tr_b16), which hands
//     lane j of a 16-lane group the four k-values of column j.
// Rows or columns beyond the tile's extent are clamped to a valid one (they only reach outputs that are never
// stored), reduction indices beyond K are zeros in both operands (load_edge).
constexpr int BM = 256, BN = 256, BK = 64;
constexpr int GT = 256;

__device__ __attribute__((aligned(16))) uint16_t g_zero_chunk[8] = {0, 0, 0, 0, 0, 0, 0, 0};

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short shortx4;
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int intx4;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned uintx4;
typedef __attribute__((__vector_size__(2 * sizeof(unsigned)))) unsigned uintx2;
// Byte offset outside every buffer descriptor of this file (and its length): a load there gives zeros, a store is
// dropped.  Valid offsets stay under 2^32 - 8192, the biases of the loads included.
constexpr unsigned OUTSIDE = 0xfffff000u;
#define SYMI_GPTR(p) ((const void __attribute__((address_space(1)))*)(p))
#define SYMI_LPTR(p) ((void __attribute__((address_space(3)))*)(p))

__device__ __forceinline__ void wait_vmcnt0() { __builtin_amdgcn_s_waitcnt(0x0F70); }

template <int V> struct IC { static constexpr int value = V; };
template <int N, int I = 0, class F>
__device__ __forceinline__ void unroll(F&& f) {   // f(IC<0>{}) .. f(IC<N - 1>{})
  if constexpr (I < N) {
    f(IC<I>{});
    unroll<N, I + 1>(f);
  }
}

// LDS reads with an immediate byte offset; nothing waits for them (see the kernel)
template <int OFF>
__device__ __forceinline__ bf16x8 lds_read_b128(unsigned addr) {
  bf16x8 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
  return v;
}
// transposing read: 4 k-values of one column per 8-byte half; the second half sits 4 k-rows
// (2048 bytes) further
template <int OFF>
__device__ __forceinline__ bf16x8 lds_read_tr(unsigned addr) {
  shortx4 lo, hi;
  asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
               : "=&v"(lo), "=&v"(hi) : "v"(addr), "n"(OFF), "n"(OFF + 2048));
  union { shortx4 h[2]; bf16x8 v; } u;
  u.h[0] = lo;
  u.h[1] = hi;
  return u.v;
}

// acc += b * a, the accumulator pinned to AGPRs: through the builtin the register allocator moved
// accumulators between the two halves of the register file inside the loop (about 600 moves per 256 MFMAs)
__device__ __forceinline__ void mfma_acc(floatx4& acc, bf16x8 b, bf16x8 a) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(b), "v"(a));
}

// Reduction slices of the narrow variable-row products (FWD2, BWD_DX).  Their tiles run in
// launch order, one workgroup per tile, in rounds of `cus`.  If the last round would leave at
// least half the chip idle (config c2: 300 tiles, a second round of 44), each of its tiles is
// cut into `sl` slices of at least 16 reduction steps, as many as fill the round (at most 8);
// a slice leaves its accumulators as a plain fp32 tile in a partial slot and slice_sum_kernel,
// launched behind the product, adds them up in slice order.  full = tiles that stay whole.
// (Letting the slice that finishes last add up the partials inside the product was measured
// slower than no slicing at all: device-scope fences write back / invalidate the whole L2 of
// an XCD under the other tiles' feet, and without fences one workgroup reads a megabyte of
// uncached partials at some 16 GB/s.  Slicing the weight gradients of very popular classes the
// same way cost more in partial traffic than the shorter tail returned.)
__device__ __forceinline__ void tail_slices(int n_tiles, int cus, int K, int& full, int& sl) {
  full = n_tiles;
  sl = 1;
  const int rem = n_tiles % cus;
  if (rem > 0 && 2 * rem <= cus) {
    const int s = min(min(cus / rem, 8), (K + BK - 1) / BK / 16);
    if (s >= 2) { sl = s; full = n_tiles - rem; }
  }
}

// Saved u, v of a wavefront's 32-row block, for the epilogue of the hidden gradient.
template <int NJ>
struct SavedUV { uint4 u[NJ * 2], v[NJ * 2]; };

// The loads are unconditional: a lane past the tile's last row or column reads the last valid row / the last 8
// columns instead (its result is never stored).  A load under a branch would make the compiler lose count of the
// memory operations in flight and wait for all of them, the stores of the previous rows included, before every
// use of a loaded value.
template <int NJ>
__device__ __forceinline__ void load_uv(const GemmParams& p, const int rb, const int row1, const int c0, const int lane,
                                        SavedUV<NJ>& s) {
  constexpr int LB = 4 * NJ;   // lanes that share a row
  const int twof = 2 * p.f, colc = min(c0 + (lane & (LB - 1)) * 8, p.N - 8);
  const uint16_t* const q0 = static_cast<const uint16_t*>(p.UV) + (long long)rb * twof + colc;
#pragma unroll
  for (int it = 0; it < 2 * NJ; ++it) {
    const int dr = min(rb + it * (64 / LB) + lane / LB, row1 - 1) - rb;   // may be negative
    const uint16_t* const q = q0 + (long long)dr * twof;
    s.u[it] = *reinterpret_cast<const uint4*>(q);
    s.v[it] = *reinterpret_cast<const uint4*>(q + p.f);
  }
}

// Epilogue of a tile whose wavefronts own 32 MI x 32 NJ outputs each.  After the MFMA a lane owns
// one output row (lane%16) of each 16 x 16 block and its 4 columns 4*(lane/16) ..: stored like that,
// a wavefront store would touch 16 cache lines with 64 or 32 bytes each, and the store path is
// paid per line touched.  The operand stages are free now, so every wavefront turns its
// 32-row blocks around through a private piece of LDS (`stg`; written in the MFMA layout, read
// back row by row, 16 bytes per lane) and each store instruction writes whole lines: for NJ = 4
// 4 rows x 256 B (bf16 outputs), 8 rows x 128 B (u, v, h) or 2 rows x 512 B (fp32).
// pslot >= 0: the accumulators of a reduction slice, left as an fp32 tile in that partial slot.
// BWD_DH: saved[0] holds (or is about to receive) the saved u, v of the first 32-row block.
template <int MODE, int MI, int NJ>
__device__ __forceinline__ void write_tile(const GemmParams& p, uint16_t* const stg, floatx4 (&acc)[2 * MI][2 * NJ],
                                           const int row0, const int row1, const int group, const int n0,
                                           const int wm, const int wn, const int lane, const int pslot,
                                           SavedUV<NJ> (&saved)[2]) {
  constexpr bool VARM = MODE <= BWD_DX;
  constexpr int WROWS = 32 * MI;
  constexpr int CW = 32 * NJ, UW = 16 * NJ;   // columns of a wavefront; FWD1: its hidden units
  constexpr int LB = CW / 8, LF = CW / 4, LH = UW / 8;   // lanes that share a row of 16-byte pieces
  const int hq = lane >> 4, r16 = lane & 15;
  constexpr int LDB = CW + 8;   // bf16 row + pad (a multiple of 16 bytes)
  constexpr int LDH = UW + 8;   // u / v / h rows + pad
  constexpr int LDF = CW + 4;   // fp32 row + pad
  constexpr int NUV = 32 / (64 / LB);
  // a slice stores its accumulators the way a weight gradient is stored: fp32, pitch 256
  const bool to_partial = (MODE == FWD2 || MODE == BWD_DX) && pslot >= 0;
  // Lanes past the tile's last row or column store to an offset outside the buffer, which drops the store: a branch
  // around every store kept the compiler from reading the staged rows ahead of it, and every 1 KB stored waited for
  // an LDS round trip of its own.
  auto store16 = [&](void* ubase, bool in, unsigned ofs, uint4 x) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(ubase, 0, (int)OUTSIDE, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, x), rsrc, (int)(in ? ofs : OUTSIDE), 0, 0);
  };
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    const int rbase = row0 + wm * WROWS + i * 32;   // first output row of this block
    const int left = row1 - rbase;                  // rows from there on
    if (MODE == FWD1) {
      uint16_t* const su = stg;
      uint16_t* const sv = stg + 32 * LDH;
      uint16_t* const sh = stg + 64 * LDH;
#pragma unroll
      for (int ih = 0; ih < 2; ++ih)
#pragma unroll
        for (int q = 0; q < NJ; ++q) {   // 16 hidden units
          const int g = 4 * (q >> 1) + (q & 1);
          unsigned pu[2], pv[2], ph[2];
#pragma unroll
          for (int c2 = 0; c2 < 2; ++c2) {
            float u0 = acc[2 * i + ih][g][2 * c2], u1 = acc[2 * i + ih][g][2 * c2 + 1];
            float v0 = acc[2 * i + ih][g + 2][2 * c2], v1 = acc[2 * i + ih][g + 2][2 * c2 + 1];
            // one read of each accumulator: the compiler would rather fetch it from its AGPR again for every use
            asm("" : "+v"(u0), "+v"(u1), "+v"(v0), "+v"(v1));
            pu[c2] = pack_bf16x2(u0, u1);
            pv[c2] = pack_bf16x2(v0, v1);
            ph[c2] = pack_bf16x2(u0 * sigmoid_fast(u0) * v0, u1 * sigmoid_fast(u1) * v1);
          }
          const int at = (ih * 16 + r16) * LDH + 16 * q + 4 * hq;
          *reinterpret_cast<uint2*>(su + at) = make_uint2(pu[0], pu[1]);
          *reinterpret_cast<uint2*>(sv + at) = make_uint2(pv[0], pv[1]);
          *reinterpret_cast<uint2*>(sh + at) = make_uint2(ph[0], ph[1]);
        }
      asm volatile("" ::: "memory");   // a wavefront's LDS operations are carried out in order
      uint16_t* const UVo = static_cast<uint16_t*>(p.UVout) + (long long)rbase * 2 * p.f;
      uint16_t* const Ho = static_cast<uint16_t*>(p.H) + (long long)rbase * p.f;
      const int hu = n0 + wn * UW + (lane & (LH - 1)) * 8;
      constexpr int NIT = 32 * LH / 64;
      uint4 xu[NIT], xv[NIT], xh[NIT];
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int at = (it * (64 / LH) + lane / LH) * LDH + (lane & (LH - 1)) * 8;
        xu[it] = *reinterpret_cast<const uint4*>(su + at);
        xv[it] = *reinterpret_cast<const uint4*>(sv + at);
        xh[it] = *reinterpret_cast<const uint4*>(sh + at);
      }
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int rr = it * (64 / LH) + lane / LH;
        const bool in = rr < left && hu < p.f;
        const unsigned o = (unsigned)(rr * p.f + hu) * 2u;
        store16(UVo, in, o + (unsigned)(rr * p.f) * 2u, xu[it]);
        store16(UVo + p.f, in, o + (unsigned)(rr * p.f) * 2u, xv[it]);
        store16(Ho, in, o, xh[it]);
      }
    } else if (MODE == BWD_DH) {
      // dh stays in fp32: staged like a weight-gradient block, then every lane takes 8
      // consecutive hidden units of one row, combines them with the saved u and v (16 bytes
      // each, whole lines per instruction) and writes du = dh v s (1 + u (1 - s)),
      // dv = dh u s, s = sigmoid(u).  The u, v loads of block i + 1 are issued before block i
      // is worked on, those of the first block before the last reduction steps, so their latency is hidden.
      float* const sf = reinterpret_cast<float*>(stg);
      uint16_t* const Co = static_cast<uint16_t*>(p.C) + (long long)rbase * 2 * p.f;
      const int col = n0 + wn * CW + (lane & (LB - 1)) * 8;
      const int twof = 2 * p.f;
      if (i + 1 < MI) load_uv<NJ>(p, row0 + wm * WROWS + (i + 1) * 32, row1, n0 + wn * CW, lane, saved[(i + 1) & 1]);
#pragma unroll
      for (int ih = 0; ih < 2; ++ih)
#pragma unroll
        for (int j = 0; j < 2 * NJ; ++j)
          *reinterpret_cast<floatx4*>(sf + (ih * 16 + r16) * LDF + 16 * j + 4 * hq) = acc[2 * i + ih][j];
      asm volatile("" ::: "memory");
#pragma unroll
      for (int it = 0; it < NUV; ++it) {
        const int rr = it * (64 / LB) + lane / LB;
        const float4 d0 = *reinterpret_cast<const float4*>(sf + rr * LDF + (lane & (LB - 1)) * 8);
        const float4 d1 = *reinterpret_cast<const float4*>(sf + rr * LDF + (lane & (LB - 1)) * 8 + 4);
        const bool in = rr < left && col < p.N;
        const unsigned o = (unsigned)(rr * twof + col) * 2u;
        const uint4 uu = saved[i & 1].u[it], vv = saved[i & 1].v[it];
        const float dh[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
        const uint32_t uw[4] = {uu.x, uu.y, uu.z, uu.w}, vw[4] = {vv.x, vv.y, vv.z, vv.w};
        uint32_t du[4], dv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float o_du[2], o_dv[2];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const float u_ = __uint_as_float(h ? (uw[q] & 0xffff0000u) : (uw[q] << 16));
            const float v_ = __uint_as_float(h ? (vw[q] & 0xffff0000u) : (vw[q] << 16));
            const float sg = sigmoid_fast(u_);
            // dh v and dh u first: dh s is subnormal, a few bits long, for u near -87 and small dh
            o_du[h] = dh[2 * q + h] * v_ * sg * (1.f + u_ * (1.f - sg));
            o_dv[h] = dh[2 * q + h] * u_ * sg;
          }
          du[q] = pack_bf16x2(o_du[0], o_du[1]);
          dv[q] = pack_bf16x2(o_dv[0], o_dv[1]);
        }
        store16(Co, in, o, make_uint4(du[0], du[1], du[2], du[3]));
        store16(Co + p.f, in, o, make_uint4(dv[0], dv[1], dv[2], dv[3]));
      }
    } else if ((MODE == FWD2 || MODE == BWD_DX) && !to_partial) {
#pragma unroll
      for (int ih = 0; ih < 2; ++ih)
#pragma unroll
        for (int j = 0; j < 2 * NJ; ++j) {
          const floatx4 x = acc[2 * i + ih][j];
          *reinterpret_cast<uint2*>(stg + (ih * 16 + r16) * LDB + 16 * j + 4 * hq) =
              make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
        }
      asm volatile("" ::: "memory");
      uint16_t* const Co = static_cast<uint16_t*>(p.C) + (long long)rbase * p.N;
      const int col = n0 + wn * CW + (lane & (LB - 1)) * 8;
      uint4 x[NUV];
#pragma unroll
      for (int it = 0; it < NUV; ++it)
        x[it] = *reinterpret_cast<const uint4*>(stg + (it * (64 / LB) + lane / LB) * LDB + (lane & (LB - 1)) * 8);
#pragma unroll
      for (int it = 0; it < NUV; ++it) {
        const int rr = it * (64 / LB) + lane / LB;
        store16(Co, rr < left && col < p.N, (unsigned)(rr * p.N + col) * 2u, x[it]);
      }
    } else {   // weight gradients, fp32
      float* const sf = reinterpret_cast<float*>(stg);
#pragma unroll
      for (int ih = 0; ih < 2; ++ih)
#pragma unroll
        for (int j = 0; j < 2 * NJ; ++j)
          *reinterpret_cast<floatx4*>(sf + (ih * 16 + r16) * LDF + 16 * j + 4 * hq) = acc[2 * i + ih][j];
      asm volatile("" ::: "memory");
      constexpr int NIT = 32 * LF / 64;
      uint4 x[NIT];
#pragma unroll
      for (int it = 0; it < NIT; ++it)
        x[it] = *reinterpret_cast<const uint4*>(sf + (it * (64 / LF) + lane / LF) * LDF + (lane & (LF - 1)) * 4);
      if (VARM) {   // a slice's partial tile
        float* Co = p.partials + (size_t)pslot * (BM * BN) + (wm * WROWS + i * 32) * BN + wn * CW + (lane & (LF - 1)) * 4;
#pragma unroll
        for (int it = 0; it < NIT; ++it) *reinterpret_cast<uint4*>(Co + (it * (64 / LF) + lane / LF) * BN) = x[it];
      } else {
        float* const Co = static_cast<float*>(p.C) + (long long)group * p.c_group_stride + (long long)rbase * p.N;
        const int col = n0 + wn * CW + (lane & (LF - 1)) * 4;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
          const int rr = it * (64 / LF) + lane / LF;
          store16(Co, rr < left && col < p.N, (unsigned)(rr * p.N + col) * 4u, x[it]);
        }
      }
    }
    // the next block reuses the staging area: its writes must not pass these reads
    asm volatile("" ::: "memory");
  }
}

// One tile of one product.  MI = 32-row blocks per wavefront: 4 for the 256-row tile (each of the
// 2 x 2 wavefronts 128 x 128), 2 for the 128-row tile that holds the ragged end of a slot when
// it has at most 128 rows (each wavefront 64 x 128: half the MFMAs, and the two wavefronts whose
// 64-row band of the left operand lies beyond the tile load nothing of it).
template <int MODE, int MI>
__device__ __forceinline__ void gemm_tile(const GemmParams& p, uint16_t* const smem, const int row0,
                                          const int row1, const int group, const int kbeg, const int K,
                                          const int bx, const int nsl, const int kofs, const int pslot) {
  // [left stages 0, 1 | right stages 0, 1, 2], 32 KB each: the two left stages differ by an immediate
  // offset of the LDS read instructions, the addresses of the right operand move on with every step
  uint16_t* const sA0 = smem;
  uint16_t* const sA1 = smem + BM * BK;
  uint16_t* const sB0 = smem + 2 * BM * BK;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, and known to be
  const int wm = wave >> 1, wn = wave & 1;
  constexpr bool VARM = MODE <= BWD_DX;
  constexpr bool A_KC = VARM;                       // left operand reduction-contiguous
  constexpr bool B_KC = MODE == FWD1 || MODE == FWD2;
  constexpr int WROWS = 32 * MI;                    // output rows of one wavefront
  static_assert(MI == 4 || (MI == 2 && VARM), "the 128-row tile serves the variable-row products");
  // a wavefront whose 64 rows of the left tile lie beyond a 128-row tile loads nothing of it
  const bool skip_left = MI == 2 && wave >= 2;
  // FWD1: a tile holds 128 hidden units; every 64 tile columns are 32 gate columns
  // followed by the 32 up columns of the same hidden units.
  const int n0 = bx * (MODE == FWD1 ? BN / 2 : BN);

  if (!VARM && K == 0) {
    if (p.skip_empty) return;   // the caller treats this gradient as zero without reading it
    // a class without rows: its gradient tile is zero; stream it out with one 1 KB row
    // segment per wavefront store
    float* Co = static_cast<float*>(p.C) + (long long)group * p.c_group_stride;
    const int col = n0 + lane * 4;
    if (col < p.N) {
      for (int r = row0 + wave; r < row1; r += GT / 64)
        *reinterpret_cast<float4*>(Co + (long long)r * p.N + col) = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    return;
  }

  const uint16_t* A = static_cast<const uint16_t*>(p.A);
  const uint16_t* B = static_cast<const uint16_t*>(p.B) + (VARM ? (long long)group * p.b_group_stride : 0);
  const long long lda = MODE == FWD1 ? p.d : MODE == FWD2 ? p.f : MODE == BWD_DH ? p.d
                        : MODE == BWD_DX ? 2LL * p.f : MODE == WGRAD2 ? p.d : 2LL * p.f;
  const long long ldb = MODE == FWD1 ? p.d : MODE == FWD2 ? p.f : MODE == BWD_DH ? p.f
                        : MODE == BWD_DX ? p.d : MODE == WGRAD2 ? p.f : p.d;

  // ---- direct-to-LDS loads: a wave-uniform base per reduction step plus a 32-bit per-lane
  // element offset, one per instruction j (0..7) and operand.
  // reduction-contiguous tile: wavefront w, instruction j fills tile rows w*64 + 8j .. +8;
  //   lane -> (row + lane/8, physical chunk lane%8)
  // reduction-strided tile: wavefront w, instruction j fills k-rows w*16 + 2j, +1;
  //   lane -> (k-row + lane/32, physical chunk lane%32)
  // Rows / column chunks beyond the operand's extent are clamped to a valid one: what
  // they bring in only reaches outputs that are never stored.
  // The 16 offsets stay in registers (no vector arithmetic next to the MFMAs).
  const int kc_row = wave * 64 + (lane >> 3);                  // tile row of instruction 0
  const int kc_c0 = (lane & 7) ^ ((lane >> 4) & 7);            // logical chunk for even j
  const int ks_kb = wave * 16 + (lane >> 5);                   // k-row of instruction 0
  const int ks_c0 = (lane & 31) ^ (10 * (lane >> 5));          // logical chunk, j-dependent bits to come
  const int f1_row = wave * 32 + (lane >> 3);                  // FWD1 weights: hidden unit of instruction 0

  const uint16_t* a_base;   // element (first tile row / column, reduction index 0)
  const uint16_t* b_base;
  int a_lim, b_lim;         // KC: last valid tile row; KS: number of valid columns
  if (A_KC) {
    a_base = A + (long long)row0 * lda + kofs;
    a_lim = row1 - row0 - 1;
  } else {
    a_base = A + (long long)kbeg * lda + row0;
    a_lim = row1 - row0;
  }
  if (B_KC) {
    b_base = (MODE == FWD1 ? B : B + (long long)n0 * ldb) + kofs;
    b_lim = MODE == FWD1 ? p.f - 1 : p.N - n0 - 1;
  } else {
    b_base = (VARM ? B + (long long)kofs * ldb : B + (long long)kbeg * ldb) + n0;
    b_lim = p.N - n0;
  }
  // LDS destination of instruction j (wave-uniform): both layouts advance 1 KB per j
  const int wdst = wave * 8 * 512;  // elements: 8 instructions x 512 elements per wavefront
  // q = 0..15: even = left operand, odd = right operand, instruction j = q/2
  // offset of this lane's 16 bytes for instruction j
  auto lane_off = [&](bool right, int j) -> unsigned {
    const bool kcontig = right ? B_KC : A_KC;
    const int ld = (int)(right ? ldb : lda);
    const int lim = right ? b_lim : a_lim;
    if (kcontig) {
      const int kc = kc_c0 ^ (4 * (j & 1));
      if (right && MODE == FWD1) {
        // tile row t -> hidden unit n0 + (t>>7)*64 + ((t>>6)&1)*32 + (t&31), up half if (t>>5)&1
        const int hu = min(n0 + f1_row + 8 * (j & 3), lim);
        return (unsigned)(((j >> 2) * p.f + hu) * ld + kc * 8);
      }
      return (unsigned)(min(kc_row + 8 * j, lim) * ld + kc * 8);
    }
    const int c = ks_c0 ^ (4 * (j & 1)) ^ (2 * ((j >> 2) & 1));
    return (unsigned)((ks_kb + 2 * j) * ld + (c * 8 < lim ? c : 0) * 8);
  };
  // The main loop's loads take the cheapest form the instruction has: a scalar base (operand +
  // reduction step), a 32-bit per-lane byte offset from a register and an immediate, with the
  // LDS base (M0) written once per operand and stage: the 8 instructions of an operand write 8
  // consecutive KB, reached from an M0 in their middle through immediates of -4 .. +3 KB, which
  // the per-lane offset takes back out of the global address (the scalar base sits 4 KB low so
  // that the offset stays positive).  Measured in the loop's microbenchmark: an M0 write in front
  // of every load and a 64-bit vector add for its address cost 26-36 cycles of MFMA issue per
  // load, this form 4-8 (a 64-deep step 2750 -> 2340 cycles).  All direct-to-LDS loads of this
  // kernel are inline assembly, so that nothing else ever writes M0.
  unsigned voA[8], voB[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    voA[j] = lane_off(false, j) * 2u + 4096u - (unsigned)((j - 4) * 1024);
    voB[j] = lane_off(true, j) * 2u + 4096u - (unsigned)((j - 4) * 1024);
  }
  // a direct-to-LDS load needs one wait state behind a write of M0, and the compiler, which would put it
  // there, does not look inside inline assembly
  auto set_m0 = [&](unsigned lds_byte_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" ::"s"(lds_byte_addr) : "memory");
  };
  auto load_fast = [&](auto jc, unsigned voff, const void* sbase) {
    constexpr int J = decltype(jc)::value;
    asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(voff), "s"(sbase), "n"((J - 4) * 1024) : "memory");
  };
  // The last pairs of steps, which load indices beyond K, take the buffer form of the load: a lane whose
  // offset lies outside the buffer gets zeros, so a ragged end costs a compare and a select per load.  (With
  // 64-bit addresses, recomputed per load, and those lanes pointed at a block of zeros in memory, such a step took
  // 3600 cycles against 2390 of a full one of c4's first forward product, and an odd step count a whole idle step more: 14400
  // cycles of 46000 for a tile of per-slot gradients, K = 384 on average.  Same bits; step E = 64, d = 2048, f = 1408 with
  // per-slot gradients of 49152 rows 3727 -> 3581 us, backward of E = 12, d = 1160, f = 2744, 15009 rows 871 -> 855, c4
  // 10.39 -> 10.27 ms.)  The immediate is unsigned here: the eight instructions of an operand take two M0 values and
  // two bases 4 KB apart.
  auto load_edge = [&](auto jc, unsigned voff, const char* base) {
    constexpr int J = decltype(jc)::value;
    const unsigned long long a = (unsigned long long)(base - (J < 4 ? 4096 : 0));
    const intx4 rsrc = {(int)(unsigned)a, (int)((unsigned)(a >> 32) & 0xffffu), (int)OUTSIDE, 0x00020000};
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen offset:%2 lds" ::"v"(voff), "s"(rsrc), "n"((J & 3) * 1024) : "memory");
  };
  // q = 0..7: instruction j = q of the left operand, q = 8..15: instruction j = q - 8 of the right one
  auto dma_one = [&](unsigned lds_stage, int k0, auto qc, auto partial) {
    constexpr int Q = decltype(qc)::value;
    constexpr int j = Q & 7;
    constexpr bool right = Q >= 8;
    if (MI == 2 && !right && skip_left) return;
    const bool kcontig = right ? B_KC : A_KC;
    const uint16_t* base = right ? b_base : a_base;
    const long long ld = right ? ldb : lda;
    const uint16_t* sbase = kcontig ? base + k0 : base + (long long)k0 * ld;   // wave-uniform
    const unsigned lds0 = lds_stage + 2 * wdst;   // this wavefront's 8 KB of the stage
    if (decltype(partial)::value) {
      const int left = K - k0;   // reduction indices of this step; a multiple of 8 where they are contiguous
      const bool in = kcontig ? (kc_c0 ^ (4 * (j & 1))) < (left >> 3) : ks_kb < left - 2 * j;
      if (j == 0) set_m0(lds0);
      if (j == 4) set_m0(lds0 + 4096);
      load_edge(IC<j>{}, in ? (right ? voB[j] : voA[j]) : OUTSIDE, reinterpret_cast<const char*>(sbase) - 4096);
    } else {
      if (j == 0) set_m0(lds0 + 4096);
      load_fast(IC<j>{}, right ? voB[j] : voA[j], reinterpret_cast<const char*>(sbase) - 4096);
    }
  };
  // ---- fragment reads.  Byte address of this lane's piece inside stage 0 of its operand,
  // everything else (16-row block, 32-deep sub-step, left stage) is an immediate offset.
  // KC: row (block*16 + lane%16), chunk (4*ks + lane/16) ^ ((lane%16 >> 1) & 7); the xor makes the
  //   sub-step a per-lane quantity, so there is one address per sub-step.
  // KS: lane = 16*g + jj supplies the address of k-row (32*ks + 8*g + 4*e + jj/4), 8-byte piece (jj%4)
  //   of the block's 16 columns; it receives column block*16 + jj; one address per block, the
  //   sub-step is an immediate (32 k-rows of 512 B).
  const int g4 = lane >> 4, jj = lane & 15;
  const int ks_h = (10 * ((jj >> 2) & 1)) ^ (4 * ((jj >> 3) & 1)) ^ (2 * (g4 & 1));   // swizzle of this lane's k-row
  const int ks_row = (8 * g4 + (jj >> 2)) * 256;
  unsigned adA[A_KC ? 2 : 2 * MI], adB[B_KC ? 2 : 8];
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    const int kc = jj * BK + (((4 * x + g4) ^ ((jj >> 1) & 7)) * 8);                                // x = sub-step
    const int ksc = ks_row + (((2 * x + ((jj & 3) >> 1)) ^ ks_h) * 8) + 4 * (jj & 1);               // x = block
    if (x < (A_KC ? 2 : 2 * MI)) adA[x] = (unsigned)(size_t)SYMI_LPTR(sA0) + 2u * (unsigned)(A_KC ? wm * WROWS * BK + kc : wm * WROWS + ksc);
    if (x < (B_KC ? 2 : 8)) adB[x] = (unsigned)(size_t)SYMI_LPTR(sB0) + 2u * (unsigned)(B_KC ? wn * 128 * BK + kc : wn * 128 + ksc);
  }
  // All LDS reads are inline assembly: the compiler cannot tell the stage being read from the
  // one being filled by direct-to-LDS loads and would wait for the prefetch before every
  // read.  Completion is awaited by hand (lgkmcnt(0)) at the start of the phase that uses them.
  // Two register sets each: one feeds the MFMAs, the other is being filled.  fa holds the left operand's
  // blocks of a phase (half of the wavefront's rows), fb the right operand's of a sub-step.
  bf16x8 fa[2][MI], fb[2][8];
  auto read_a = [&](auto setc, auto stagec, auto ksc, auto halfc, auto qc) {
    constexpr int SO = decltype(stagec)::value * BM * BK * 2, KS = decltype(ksc)::value;   // stage offset in bytes
    constexpr int q = decltype(qc)::value, blk = decltype(halfc)::value * MI + q;
    if constexpr (A_KC) fa[decltype(setc)::value][q] = lds_read_b128<SO + blk * 2048>(adA[KS]);
    else fa[decltype(setc)::value][q] = lds_read_tr<SO + KS * 16384>(adA[blk]);
  };
  auto read_b = [&](auto ksc, auto jc) {
    constexpr int KS = decltype(ksc)::value, j = decltype(jc)::value;
    if constexpr (B_KC) fb[KS][j] = lds_read_b128<j * 2048>(adB[KS]);
    else fb[KS][j] = lds_read_tr<KS * 16384>(adB[j]);
  };
  const unsigned ldsA0 = (unsigned)(size_t)SYMI_LPTR(sA0), ldsA1 = (unsigned)(size_t)SYMI_LPTR(sA1);
  const unsigned ldsB = (unsigned)(size_t)SYMI_LPTR(sB0);
  int bs = 0;   // byte offset of the right operand's stage of this step (adB points into it)

  floatx4 acc[2 * MI][8];
#pragma unroll
  for (int i = 0; i < 2 * MI; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // ---- main loop.  A reduction step (64 deep, left stage S = step & 1, right stage step % 3) is four
  // phases of 32 MFMAs: sub-step 0 and 1, in each the upper and the lower half of the wavefront's rows.
  // A phase reads the fragments of the next one into the other register set.  Phase 3 first waits for
  // the loads of the next step and meets the other wavefronts, after which nobody reads this step's
  // stages any more (their last fragments already sit in registers); it reads the first fragments of
  // the next stages.  Phases 3 and 0 load the left operand of step + 2 into the stage just freed, phases 1
  // and 2 the right one of step + 2 into the stage freed a step ago.  Neither an LDS round trip nor a load
  // latency is exposed to the MFMA pipe.  Steps beyond the last one load zeros (dummy
  // loads keep the loop free of branches).
  const int nk = (K + BK - 1) / BK;
  auto phase = [&](auto ksc, auto stagec, int step, auto partial) {
    constexpr int KS = decltype(ksc)::value, S = decltype(stagec)::value;
    constexpr int half = KS & 1, sub = KS >> 1;
    const unsigned cA = S ? ldsA1 : ldsA0, oA = S ? ldsA0 : ldsA1;
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the fragments of this phase
    if (KS == 3) {
      __builtin_amdgcn_s_waitcnt(0x0F78);   // my share of the next step has landed (the 8 loads of the step after it may fly)
      __builtin_amdgcn_s_barrier();       // ... so has everybody's, and stage S is free
    }
    __builtin_amdgcn_sched_barrier(0);
    constexpr int NB = KS == 0 || KS == 1 ? 4 : KS == 2 ? 0 : 8;   // right blocks read in this phase
    auto read = [&](auto rc) {
      constexpr int r = decltype(rc)::value;
      if constexpr (r < MI) {
        if constexpr (KS == 0) read_a(IC<1>{}, IC<S>{}, IC<0>{}, IC<1>{}, IC<r>{});
        if constexpr (KS == 1) read_a(IC<0>{}, IC<S>{}, IC<1>{}, IC<0>{}, IC<r>{});
        if constexpr (KS == 2) read_a(IC<1>{}, IC<S>{}, IC<1>{}, IC<1>{}, IC<r>{});
        if constexpr (KS == 3) read_a(IC<0>{}, IC<S ^ 1>{}, IC<0>{}, IC<0>{}, IC<r>{});
      } else if constexpr (r < MI + NB) {
        if constexpr (KS == 0) read_b(IC<1>{}, IC<r - MI>{});
        if constexpr (KS == 1) read_b(IC<1>{}, IC<r - MI + 4>{});
        if constexpr (KS == 3) read_b(IC<0>{}, IC<r - MI>{});
      }
    };
    constexpr int RS = MI == 4 ? 2 : 1, LS = 2 * MI, L0 = MI == 4 ? 5 : 1;   // every RS-th MFMA a read, every LS-th a load
    unroll<8 * MI>([&](auto mc) {
      constexpr int m = decltype(mc)::value, i = m >> 3, j = i & 1 ? 7 - (m & 7) : m & 7;
      mfma_acc(acc[half * MI + i][j], fb[sub][j], fa[half][i]);
      if constexpr (m % RS == 0) read(IC<m / RS>{});
      // phases 3 and 0: the left operand of step + 2 into the stage freed at this phase 3; phases 1 and 2: the right one
      constexpr int L = m >= L0 && (m - L0) % LS == 0 ? (m - L0) / LS : 4;
      if constexpr (L < 4) {
        if constexpr (KS == 3) dma_one(cA, (step + 2) * BK, IC<L>{}, partial);
        if constexpr (KS == 0) dma_one(oA, (step + 1) * BK, IC<4 + L>{}, partial);
        if constexpr (KS == 1) dma_one(ldsB + (bs == 0 ? 2 * BN * BK * 2 : bs - BN * BK * 2), (step + 2) * BK, IC<8 + L>{}, partial);
        if constexpr (KS == 2) dma_one(ldsB + (bs == 0 ? 2 * BN * BK * 2 : bs - BN * BK * 2), (step + 2) * BK, IC<12 + L>{}, partial);
      }
      if constexpr (KS == 2 && m == 8 * MI - 1) {   // on to the right operand's next stage
        const int next = bs == 2 * BN * BK * 2 ? 0 : bs + BN * BK * 2;
#pragma unroll
        for (int x = 0; x < (B_KC ? 2 : 8); ++x) adB[x] += (unsigned)(next - bs);
        bs = next;
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto pair = [&](int t, auto partial) {
    phase(IC<0>{}, IC<0>{}, t, partial);
    phase(IC<1>{}, IC<0>{}, t, partial);
    phase(IC<2>{}, IC<0>{}, t, partial);
    phase(IC<3>{}, IC<0>{}, t, partial);
    phase(IC<0>{}, IC<1>{}, t + 1, partial);
    phase(IC<1>{}, IC<1>{}, t + 1, partial);
    phase(IC<2>{}, IC<1>{}, t + 1, partial);
    phase(IC<3>{}, IC<1>{}, t + 1, partial);
  };
  auto prologue = [&](auto partial) {
    unroll<16>([&](auto q) { dma_one(decltype(q)::value < 8 ? ldsA0 : ldsB, 0, q, partial); });                              // step 0
    unroll<8>([&](auto q) { dma_one(ldsB + BN * BK * 2, BK, IC<8 + decltype(q)::value>{}, partial); });     // step 1, right operand
    unroll<4>([&](auto q) { dma_one(ldsA1, BK, q, partial); });     // and half of the left one (the rest follows in phase 0)
  };
  if (K >= 2 * BK) prologue(std::false_type{}); else prologue(std::true_type{});
  // step 0 has landed, the 12 loads of step 1 may still fly (8 in a wavefront of a half-height tile that
  // skips the left operand)
  if (MI == 4) __builtin_amdgcn_s_waitcnt(0x0F7C); else __builtin_amdgcn_s_waitcnt(0x0F78);
  __builtin_amdgcn_s_barrier();
  unroll<MI>([&](auto q) { read_a(IC<0>{}, IC<0>{}, IC<0>{}, IC<0>{}, q); });
  unroll<8>([&](auto q) { read_b(IC<0>{}, q); });
  // steps in pairs, an odd last one by itself; a pair starting at step t loads steps up to t + 3
  int t = 0;
  for (; (t + 4) * BK <= K; t += 2) pair(t, std::false_type{});
  SavedUV<4> saved[2];
  if (MODE == BWD_DH) load_uv<4>(p, row0 + wm * WROWS, row1, n0 + wn * 128, lane, saved[0]);
  for (; t + 1 < nk; t += 2) pair(t, std::true_type{});
  if (t < nk) {
    phase(IC<0>{}, IC<0>{}, t, std::true_type{});
    phase(IC<1>{}, IC<0>{}, t, std::true_type{});
    phase(IC<2>{}, IC<0>{}, t, std::true_type{});
    phase(IC<3>{}, IC<0>{}, t, std::true_type{});
  }
  // The dummy loads and the fragments read in the last phase are still in flight.  They must not outlive
  // the workgroup's LDS allocation, and the fragments' registers stay taken until they have landed: to
  // the compiler they are written and free, and what it moved up from the epilogue into one of them
  // would be overwritten by a late read.
  __builtin_amdgcn_s_waitcnt(0xC07F);
#pragma unroll
  for (int q = 0; q < MI; ++q) asm volatile("" : "+v"(fa[0][q]));
#pragma unroll
  for (int q = 0; q < 8; ++q) asm volatile("" : "+v"(fb[0][q]));
  // the last MFMAs are through after 16 wait states; no accumulator is read before
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
  for (int i = 0; i < 2 * MI; ++i)
    asm volatile("" : "+a"(acc[i][0]), "+a"(acc[i][1]), "+a"(acc[i][2]), "+a"(acc[i][3]), "+a"(acc[i][4]),
                 "+a"(acc[i][5]), "+a"(acc[i][6]), "+a"(acc[i][7]));
  wait_vmcnt0();

  __syncthreads();   // every wavefront's dummy loads have landed, nobody reads operands any more
  // 32 KB of the operand stages per wavefront
  write_tile<MODE, MI, 4>(p, smem + wave * (16 * 1024), acc, row0, row1, group, n0, wm, wn, lane,
                                nsl > 1 ? pslot : -1, saved);
}

// Workgroups go to the eight XCDs (each with an L2 of its own) round robin in launch order:
// workgroup b runs on XCD b mod 8.  With the column index fastest an XCD would see two (ntx = 16)
// or one (ntx = 4) column tile of every m-tile, so every activation tile is fetched by four to
// eight L2s.  Instead a round of R consecutive workgroups (R / 8 per XCD, R / ntx m-tiles) is dealt
// out in blocks: XCD c takes 4 column tiles x R / 32 m-tiles, so an operand tile along either
// edge of the block is fetched by that L2 once for the whole block.  b -> tile is a permutation
// inside the round; the caller leaves rounds that are not whole in launch order.
__device__ __forceinline__ void xcd_block(int b, int ntx, int R, int& tile) {
  if (ntx != 4 && ntx != 8 && ntx != 16 && ntx != 32) return;
  const int l = b % R, c = l & 7, s = l >> 3;
  const int xn = ntx >> 2;   // XCDs side by side along the columns
  const int n = 4 * (c % xn) + (s & 3);
  const int m = (b / R) * (R / ntx) + (R >> 5) * (c / xn) + (s >> 2);
  tile = m * ntx + n;
}

template <int MODE>
__global__ __launch_bounds__(GT) void gemm_bf16_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(1024))) uint16_t smem[2 * BM * BK + 3 * BN * BK];
  constexpr bool VARM = MODE <= BWD_DX;
  int row0, row1, group, kbeg = 0, K, bx = blockIdx.x;
  // this workgroup reduces slice zsl of nsl, starting at reduction index kofs; if nsl > 1 its
  // accumulators go to partial slot pslot
  int nsl = 1, zsl = 0, kofs = 0, pslot = 0;
  if (VARM) {
    // tiles in launch order (column index fastest); the last round's tiles may be sliced
    const int ntx = gridDim.x;
    const int n_tiles = p.tile_map[0] * ntx;
    const int b = blockIdx.y * ntx + blockIdx.x;
    int full = n_tiles, sl = 1;
    if ((MODE == FWD2 || MODE == BWD_DX) && p.partials) tail_slices(n_tiles, p.cus, p.K, full, sl);
    int tile = b;
    if (ntx == 4 || ntx == 8 || ntx == 16 || ntx == 32) {
      if (b < (full & ~255)) xcd_block(b, ntx, 256, tile);
    } else if (ntx < 32) {
      // other column counts: rounds of 8 m-tiles, XCD c takes all column tiles of the round's
      // m-tile c (launch order would scatter an m-tile's columns over all eight L2s)
      const int R = 8 * ntx;
      if (b < full - full % R) {
        const int l = b % R;
        tile = (b / R * 8 + (l & 7)) * ntx + (l >> 3);
      }
    }
    if (b >= full) {
      tile = full + (b - full) / sl;
      zsl = (b - full) % sl;
      nsl = sl;
    }
    if (tile >= n_tiles) return;
    const int mt = tile / ntx;
    bx = tile - mt * ntx;
    row0 = p.tile_map[4 + 4 * mt];
    row1 = p.tile_map[4 + 4 * mt + 1];
    group = p.tile_map[4 + 4 * mt + 2];
    K = p.K;
    if (nsl > 1) {
      const int nk_all = (p.K + BK - 1) / BK;
      const int len = ((nk_all + nsl - 1) / nsl + 1) / 2 * 2 * BK;   // whole pairs of steps
      kofs = zsl * len;
      K = max(0, min(len, p.K - kofs));
      pslot = (tile - full) * nsl + zsl;
    }
  } else {
    // classes in order of decreasing row count: the long reductions start first and the
    // short (or empty, store-only) tiles fill in behind them
    group = p.per_slot ? blockIdx.z : p.class_order[blockIdx.z];
    // the tiles of one class (or slot): whole rounds of 256, 128 or 64 workgroups are dealt out
    // in blocks per XCD (a group starts on XCD 0 whenever its tile count is a multiple of 8)
    const int ntx = gridDim.x, nt = ntx * gridDim.y;
    int tile = blockIdx.y * ntx + blockIdx.x;
    const int R = nt % 256 == 0 ? 256 : nt % 128 == 0 ? 128 : nt % 64 == 0 ? 64 : 0;
    if (R) xcd_block(tile, ntx, R, tile);
    const int mt = tile / ntx;
    bx = tile - mt * ntx;
    row0 = mt * BM;
    row1 = min(p.M, row0 + BM);
    if (p.per_slot) {   // the rows of one replica slot
      kbeg = p.slot_offsets[group];
      K = p.slot_offsets[group + 1] - kbeg;
    } else {            // the rows of all replica slots of a class
      kbeg = p.slot_offsets[p.first_slot[group]];
      K = p.slot_offsets[p.first_slot[group + 1]] - kbeg;
    }
  }
  if constexpr (VARM) {
    // the ragged end of a slot: at most 128 rows take the half-height tile
    if (__builtin_amdgcn_readfirstlane(row1 - row0) <= BM / 2) {
      gemm_tile<MODE, 2>(p, smem, row0, row1, group, kbeg, K, bx, nsl, kofs, pslot);
      return;
    }
  }
  gemm_tile<MODE, 4>(p, smem, row0, row1, group, kbeg, K, bx, nsl, kofs, pslot);
}

// ---------------------------------------------------------------- forward products of a small batch
// With few rows per slot the two forward products only stream weights: a 256-column tile has one
// workgroup per compute unit, 32 - 64 KB of weights in flight, and most of its left operand's loads and MFMAs
// are padding.  Here a tile is 64 rows x 128 columns (FWD1: 64 hidden units), three stages of 24 KB, two
// workgroups per unit.  The tiles that exist are numbered a slot's one after the other, and those of one
// column tile run next to each other in time on one XCD (workgroup number mod 8), so a slot with many rows gets
// its weights through one L2 once.  As four parts of the large tiles, all first parts launched before all
// second ones, each part fetched them anew: 4096 rows in 32 of 128 slots of d = 2048, f = 1408 287 us, now 209;
// and most of the workgroups had nothing to do: 2 rows in each of 96 slots of d = 1024, f = 4096 518 -> 513.
// Operand layout, fragments and epilogue are those of the large tile.
struct SlotTile { int row0, row1, slot, bx; };

// Row tile mt and column tile bx of this workgroup, gridDim.x column tiles per row tile: in rounds of 8 row tiles, a
// column tile of all 8 on one XCD.
__device__ __forceinline__ void deal_tile(int n_tiles, int& mt, int& bx) {
  const int ntx = gridDim.x;
  mt = blockIdx.y;
  bx = blockIdx.x;
  if (ntx & 7) {
    const int b = mt * ntx + bx, round = b / (8 * ntx);
    if (8 * round + 8 <= n_tiles) {
      const int r = b - round * 8 * ntx, q = (r & 7) * ntx + (r >> 3);
      mt = 8 * round + (q & 7);
      bx = q >> 3;
    }
  }
}

// Slot q holds ceil(rows / TM) row tiles: every workgroup counts them for itself from the slot offsets, which saves the
// launch that writes a table, for about a microsecond per workgroup (few_rows_table below).  A thread counts consecutive
// slots; the one whose slots hold the workgroup's row tile finds it.
template <int TM>
__device__ __forceinline__ bool find_slot_tile(const int32_t* __restrict__ offs, int n_slots, int32_t* const found, SlotTile& out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (n_slots + GT - 1) / GT, q0 = min(tid * per, n_slots), q1 = min(q0 + per, n_slots);
  int mine = 0;
  for (int q = q0; q < q1; ++q) mine += (offs[q + 1] - offs[q] + TM - 1) / TM;
  int incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) found[wave] = incl;
  __syncthreads();
  const int n_tiles = __builtin_amdgcn_readfirstlane(found[0] + found[1] + found[2] + found[3]);
  for (int w = 0; w < wave; ++w) incl += found[w];
  int mt, bx;
  deal_tile(n_tiles, mt, bx);
  if (mt >= n_tiles) return false;
  if (mt < incl && mt >= incl - mine) {
    int i = mt - (incl - mine), q = q0;
    for (;; ++q) {
      const int n = (offs[q + 1] - offs[q] + TM - 1) / TM;
      if (i < n) break;
      i -= n;
    }
    found[4] = q;
    found[5] = offs[q] + i * TM;
    found[6] = min(offs[q] + i * TM + TM, offs[q + 1]);
  }
  __syncthreads();
  out.slot = __builtin_amdgcn_readfirstlane(found[4]);
  out.row0 = __builtin_amdgcn_readfirstlane(found[5]);
  out.row1 = __builtin_amdgcn_readfirstlane(found[6]);
  out.bx = bx;
  return true;
}

// The same from a table of two words a tile.
__device__ __forceinline__ bool read_slot_tile(const int32_t* __restrict__ map, SlotTile& out) {
  const int n_tiles = map[0];
  int mt, bx;
  deal_tile(n_tiles, mt, bx);
  if (mt >= n_tiles) return false;
  const int entry = map[4 + 2 * mt + 1];
  out.row0 = map[4 + 2 * mt];
  out.row1 = out.row0 + (entry >> 16) + 1;
  out.slot = entry & 0xffff;
  out.bx = bx;
  return true;
}

// TABLE: the row tiles come from tile_map
template <int MODE, bool TABLE>
__global__ __launch_bounds__(GT, 2) void gemm_few_rows_kernel(GemmParams p) {
  static_assert(MODE == FWD1 || MODE == FWD2 || MODE == GATE, "both operands reduction-contiguous");
  constexpr int TM = FEW_BM, TN = 128, NST = 3, LA = 2, LB = 4;   // LA, LB: 1 KB load instructions per wavefront and stage
  constexpr int SA = TM * BK, SB = TN * BK;          // elements of a stage
  __shared__ __attribute__((aligned(1024))) uint16_t smem[NST * (SA + SB)];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  __shared__ int32_t found[8];
  SlotTile tile;
  if constexpr (MODE == GATE) {   // the tokens in order; grid.x has no limit that they could reach
    tile.row0 = blockIdx.x * TM;
    tile.row1 = min(p.M, tile.row0 + TM);
    tile.slot = 0;
    tile.bx = blockIdx.y;
  } else if constexpr (TABLE) {
    if (!read_slot_tile(p.tile_map, tile)) return;
  } else if (!find_slot_tile<TM>(p.slot_offsets, p.n_slots, found, tile)) {
    return;
  }
  const int row0 = tile.row0, row1 = tile.row1, group = tile.slot, bx = tile.bx;
  const int n0 = bx * (MODE == FWD1 ? TN / 2 : TN), K = p.K, ld = p.K;
  const uint16_t* const a_base = static_cast<const uint16_t*>(p.A) + (long long)row0 * ld;
  const uint16_t* const b_base = static_cast<const uint16_t*>(p.B) + (long long)group * p.b_group_stride +
                                 (MODE == FWD1 ? 0 : (long long)n0 * ld);

  // element offset of this lane's 16 bytes for load q of a stage (rows 8q .. 8q + 7) and their reduction
  // index in the step; rows beyond the operand's extent are clamped (they only reach outputs never stored)
  auto lane_off = [&](bool right, int q, int& krel) -> unsigned {
    const int r = q * 8 + (lane >> 3);
    krel = ((lane & 7) ^ ((r >> 1) & 7)) * 8;
    if (!right) return (unsigned)(min(r, row1 - row0 - 1) * ld + krel);
    if (MODE == FWD1) {   // every 64 tile rows: 32 gate rows and the 32 up rows of the same hidden units
      const int hu = min(n0 + (r >> 6) * 32 + (r & 31), p.f - 1);
      return (unsigned)((((r >> 5) & 1) * p.f + hu) * ld + krel);
    }
    return (unsigned)(min(r, p.N - n0 - 1) * ld + krel);
  };
  unsigned vo[LA + LB];
  int kr[LA + LB];
#pragma unroll
  for (int j = 0; j < LA + LB; ++j)
    vo[j] = lane_off(j >= LA, j < LA ? wave * LA + j : wave * LB + j - LA, kr[j]);
  const unsigned ldsA = (unsigned)(size_t)SYMI_LPTR(smem) + wave * (LA * 1024);
  const unsigned ldsB = (unsigned)(size_t)SYMI_LPTR(smem + NST * SA) + wave * (LB * 1024);
  const int nk = (K + BK - 1) / BK;
  // loads of step t into stage st; reduction indices beyond K come from a block of zeros
  auto issue = [&](int t, int st) {
    const int k0 = t * BK;
    unroll<LA + LB>([&](auto jc) {
      constexpr int j = decltype(jc)::value;
      const uint16_t* const base = (j < LA ? a_base : b_base) + k0;
      const uint16_t* const src = k0 + kr[j] < K ? base + (size_t)vo[j] : g_zero_chunk;
      const unsigned dst = j < LA ? ldsA + st * (SA * 2) + j * 1024 : ldsB + st * (SB * 2) + (j - LA) * 1024;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(dst), "v"(src) : "memory");   // the wait state of an M0 write
    });
  };
  const int g4 = lane >> 4, r16 = lane & 15;
  int adA[2], adB[2];   // fragment addresses (elements) per 32-deep sub-step
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int c = ((4 * x + g4) ^ ((r16 >> 1) & 7)) * 8;
    adA[x] = (wm * 32 + r16) * BK + c;
    adB[x] = NST * SA + (wn * 64 + r16) * BK + c;
  }
  floatx4 acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < nk) issue(t, t);
  int st = 0;
  for (int t = 0; t < nk; ++t) {
    // my fragment reads of step t - 1 are through (its stage is refilled behind the barrier) and my loads
    // of step t have landed; those of the steps after it may fly
    if (t + 1 < nk) __builtin_amdgcn_s_waitcnt(0x0070 + LA + LB); else __builtin_amdgcn_s_waitcnt(0x0070);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (t + NST - 1 < nk) issue(t + NST - 1, st == 0 ? NST - 1 : st - 1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 fa[2], fb[4];
#pragma unroll
      for (int i = 0; i < 2; ++i) fa[i] = *reinterpret_cast<const bf16x8*>(smem + st * SA + adA[ks] + i * 16 * BK);
#pragma unroll
      for (int j = 0; j < 4; ++j) fb[j] = *reinterpret_cast<const bf16x8*>(smem + st * SB + adB[ks] + j * 16 * BK);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    st = st == NST - 1 ? 0 : st + 1;
  }
  if constexpr (MODE == GATE) {   // logits, fp32: a lane holds 4 neighbouring classes of a token
    float* const Lo = static_cast<float*>(p.C);
    const float* const bias = static_cast<const float*>(p.UV);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int col = n0 + wn * 64 + 16 * j + 4 * g4;
      float bb[4] = {0.f, 0.f, 0.f, 0.f};
      if (bias) {
#pragma unroll
        for (int c = 0; c < 4; ++c) bb[c] = bias[min(col + c, p.N - 1)];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = row0 + wm * 32 + 16 * i + r16;
        if (row >= row1) continue;
        float* const at = Lo + (long long)row * p.N + col;
        const float4 x = make_float4(acc[i][j][0] + bb[0], acc[i][j][1] + bb[1], acc[i][j][2] + bb[2], acc[i][j][3] + bb[3]);
        if ((p.N & 3) == 0) {
          if (col < p.N) *reinterpret_cast<float4*>(at) = x;
        } else {
          if (col < p.N) at[0] = x.x;
          if (col + 1 < p.N) at[1] = x.y;
          if (col + 2 < p.N) at[2] = x.z;
          if (col + 3 < p.N) at[3] = x.w;
        }
      }
    }
    return;
  } else {
    __syncthreads();   // nobody reads operands any more
    // 18 KB of LDS per wavefront for its 32-row block of 64 columns
    SavedUV<2> saved[2];   // the input-gradient product's
    write_tile<MODE, 1, 2>(p, smem + wave * (NST * (SA + SB) / 4), acc, row0, row1, group, n0, wm, wn, lane, -1, saved);
  }
}

// ---------------------------------------------------------------- variable-row products of few or short tiles
// Tile of 128 x 128 (FWD1: 64 hidden units), reduction step 64, two 32 KB stages, four wavefronts of 64 x 64, two
// workgroups per compute unit, which hide each other's barriers and epilogues.  A step's fragments are all read into
// registers before its MFMAs, so that its stage is refilled during them.  Bound by the latency of a tile where the
// tiles do not fill the chip (18 - 26 us of the large tile, 10 - 14 here: K = 136 - 656, 20 slots of 80 rows on average), else by
// the LDS: a 64 x 64 wavefront tile reads twice as much per MFMA as the large tile's 128 x 128.  Operand layout,
// fragments and epilogue are those of the large tile, and so are the bits.  Tried and dropped: 32-deep steps in three
// stages with three workgroups per unit (c2's first forward product 386 -> 450 us), and this tile for the weight gradients (two
// transposing reads per fragment: c4's W1 gradient 1850 -> 3190 us, per-slot gradients of 384 rows 1120 -> 1180).
// TABLE: the row tiles come from tile_map
template <int MODE, bool TABLE>
__global__ __launch_bounds__(GT, 2) void gemm_mid_kernel(GemmParams p) {
  static_assert(MODE <= BWD_DX, "left operand reduction-contiguous");
  constexpr bool B_KC = MODE == FWD1 || MODE == FWD2;
  constexpr int TM = MID_BM, TN = 128, NL = 4;   // NL: 1 KB load instructions per wavefront, operand and stage
  constexpr int SA = TM * BK, SB = TN * BK;      // elements of a stage
  __shared__ __attribute__((aligned(1024))) uint16_t smem[2 * (SA + SB)];
  __shared__ int32_t found[8];
  SlotTile tile;
  if constexpr (TABLE) {
    if (!read_slot_tile(p.tile_map128, tile)) return;
  } else {
    if (!find_slot_tile<TM>(p.slot_offsets, p.n_slots, found, tile)) return;
  }
  const int row0 = tile.row0, row1 = tile.row1, group = tile.slot, bx = tile.bx;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int n0 = bx * (MODE == FWD1 ? TN / 2 : TN), K = p.K;
  const int rows = row1 - row0, cols = p.N - n0;
  const int ldb = B_KC ? K : p.N;
  const uint16_t* const a_base = static_cast<const uint16_t*>(p.A) + (long long)row0 * K;
  const uint16_t* const b_base = static_cast<const uint16_t*>(p.B) + (long long)group * p.b_group_stride +
                                 (MODE == FWD1 ? 0 : B_KC ? (long long)n0 * ldb : (long long)n0);

  // Loads: byte offset of this lane's 16 bytes for instruction j of an operand (its immediate, j KB, taken back out)
  // and their reduction index in the step.  Rows and columns beyond the operand's extent are clamped (they only
  // reach outputs never stored), reduction indices beyond K read from outside the buffer: zeros.
  unsigned vo[2 * NL];
  int kr[2 * NL];
#pragma unroll
  for (int j = 0; j < 2 * NL; ++j) {
    const bool right = j >= NL;
    const int q = wave * NL + (j & (NL - 1));
    unsigned e;
    if (!right || B_KC) {   // rows 8q .. 8q + 7
      const int r = q * 8 + (lane >> 3);
      kr[j] = ((lane & 7) ^ ((r >> 1) & 7)) * 8;
      if (!right) {
        e = (unsigned)(min(r, rows - 1) * K + kr[j]);
      } else if (MODE == FWD1) {   // every 64 tile rows: 32 gate rows and the 32 up rows of the same hidden units
        const int hu = min(n0 + (r >> 6) * 32 + (r & 31), p.f - 1);
        e = (unsigned)((((r >> 5) & 1) * p.f + hu) * K + kr[j]);
      } else {
        e = (unsigned)(min(r, cols - 1) * K + kr[j]);
      }
    } else {   // reduction indices 4q .. 4q + 3
      kr[j] = q * 4 + (lane >> 4);
      const int c = (lane & 15) ^ (10 * (kr[j] & 1)) ^ (4 * ((kr[j] >> 1) & 1)) ^ (2 * ((kr[j] >> 3) & 1));
      e = (unsigned)(kr[j] * ldb + (c * 8 < cols ? c * 8 : 0));
    }
    vo[j] = e * 2u + 4096u - (unsigned)((j & (NL - 1)) * 1024);
  }
  const unsigned ldsA = (unsigned)(size_t)SYMI_LPTR(smem) + wave * (NL * 1024);
  const unsigned ldsB = (unsigned)(size_t)SYMI_LPTR(smem + 2 * SA) + wave * (NL * 1024);
  const int nk = (K + BK - 1) / BK;
  // a tile of at most 64 rows: the lower wavefronts have no outputs, and nobody reads the left rows they would load
  const bool idle = wave >= 2 && rows <= TM / 2;
  auto load_one = [&](auto jc, unsigned v, intx4 rsrc) {
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen offset:%2 lds" ::"v"(v), "s"(rsrc), "n"(decltype(jc)::value * 1024) : "memory");
  };
  auto load = [&](auto rightc, unsigned dst, const uint16_t* src, int left, auto edge) {
    constexpr bool right = decltype(rightc)::value != 0;
    const unsigned long long a = (unsigned long long)src - 4096;
    const intx4 rsrc = {(int)(unsigned)a, (int)((unsigned)(a >> 32) & 0xffffu), (int)OUTSIDE, 0x00020000};
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" ::"s"(dst) : "memory");   // the wait state of an M0 write
    unroll<NL>([&](auto jc) {
      constexpr int j = decltype(jc)::value, x = right ? NL + j : j;
      const unsigned v = !decltype(edge)::value || kr[x] < left ? vo[x] : OUTSIDE;
      load_one(jc, v, rsrc);
    });
  };
  auto issue = [&](int t, int st) {
    const int k0 = t * BK;
    const uint16_t* const sa = a_base + k0;
    const uint16_t* const sb = b_base + (B_KC ? (long long)k0 : (long long)k0 * ldb);
    if (k0 + BK <= K) {
      if (!idle) load(IC<0>{}, ldsA + st * (SA * 2), sa, 0, std::false_type{});
      load(IC<1>{}, ldsB + st * (SB * 2), sb, 0, std::false_type{});
    } else {
      if (!idle) load(IC<0>{}, ldsA + st * (SA * 2), sa, K - k0, std::true_type{});
      load(IC<1>{}, ldsB + st * (SB * 2), sb, K - k0, std::true_type{});
    }
  };
  // fragment addresses (elements): KC one per sub-step, KS one per 16-column block
  const int g4 = lane >> 4, jj = lane & 15;
  const int ks_h = (10 * ((jj >> 2) & 1)) ^ (4 * ((jj >> 3) & 1)) ^ (2 * (g4 & 1));
  unsigned adA[2], adB[B_KC ? 2 : 4];
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const int kc = jj * BK + (((4 * x + g4) ^ ((jj >> 1) & 7)) * 8);
    const int ks = (8 * g4 + (jj >> 2)) * TN + (((2 * (4 * wn + x) + ((jj & 3) >> 1)) ^ ks_h) * 8) + 4 * (jj & 1);
    if (x < 2) adA[x] = (unsigned)(wm * 64 * BK + kc);
    if (x < (B_KC ? 2 : 4)) adB[x] = (unsigned)(2 * SA + (B_KC ? wn * 64 * BK + kc : ks));
  }
  floatx4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  issue(0, 0);
  if (nk > 1) issue(1, 1);
  for (int t = 0; t < nk; ++t) {
    const int st = t & 1;
    // my loads of step t have landed, those of the next step may fly
    if (t + 1 >= nk) __builtin_amdgcn_s_waitcnt(0x0F70);
    else if (idle) __builtin_amdgcn_s_waitcnt(0x0F70 + NL);
    else __builtin_amdgcn_s_waitcnt(0x0F70 + 2 * NL);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    bf16x8 fa[2][4], fb[2][4];
    if (!idle) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
        for (int i = 0; i < 4; ++i) fa[ks][i] = *reinterpret_cast<const bf16x8*>(smem + adA[ks] + st * SA + i * 16 * BK);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if constexpr (B_KC) {
            fb[ks][j] = *reinterpret_cast<const bf16x8*>(smem + adB[ks] + st * SB + j * 16 * BK);
          } else {
            union { shortx4 h[2]; bf16x8 v; } u;
            auto* const q = (shortx4 __attribute__((address_space(3)))*)SYMI_LPTR(smem + adB[j] + st * SB + ks * 32 * TN);
            u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(q);
            u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(q + TN);   // 4 reduction indices further
            fb[ks][j] = u.v;
          }
        }
      }
    }
    // the fragments of this step sit in registers, in every wavefront: its stage may be filled again
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (t + 2 < nk) issue(t + 2, st);
    if (!idle) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[ks][j], fa[ks][i], acc[i][j], 0, 0, 0);
    }
  }
  if (idle) return;
  // 16 KB of LDS per wavefront
  SavedUV<2> saved[2];
  if (MODE == BWD_DH) load_uv<2>(p, row0 + wm * 64, row1, n0 + wn * 64, lane, saved[0]);
  write_tile<MODE, 2, 2>(p, smem + wave * (2 * (SA + SB) / 4), acc, row0, row1, group, n0, wm, wn, lane, -1, saved);
}

// ---------------------------------------------------------------- weight gradients of short reductions
// Tile of 128 x 256, four wavefronts of 64 x 128, 32-deep steps in three 24 KB stages, two workgroups per compute unit, so
// that one's set-up and epilogue run beside the other's.  Bound by the stores of the gradients: with a few rows
// per class the large tile writes its 256 KB behind one step's load latency with nothing beside it.  60 drawn backwards of at
// most 144 rows per class (or slot), bf16: 1.045 times as fast (0.94 - 1.17); E = 8, d = 344, f = 752, 595 rows 75 -> 65 us, E = 128,
// d = 4048, f = 1528, 1125 rows 4206 -> 3718, E = 48, d = 144, f = 3552, 320 rows in 112 slots 542 -> 485.  Its
// 64 x 128 wavefront tile reads 1.5 times as much LDS per matrix instruction, which longer reductions pay for (64 slots of 384 rows,
// d = 2048, f = 1408, W1 499 : 527).  Same bits as the large tile.  Tried and dropped for the variable-row products: with 32-deep steps a
// reduction-contiguous row is half a cache line (16 slots of 1024 rows, d = f = 4096, first forward product 807 : 1192).
// LDS: [k][row] as loaded, 32-byte piece c of row k at c ^ ((k & 3) + 4 ((k >> 3) & 1)), free of bank conflicts for transposing reads.
constexpr int DUO_BM = 128, DUO_BN = 256, DUO_BK = 32;

template <int MODE>
__global__ __launch_bounds__(GT, 2) void gemm_duo_kernel(GemmParams p) {
  static_assert(MODE >= WGRAD2, "both operands reduction-strided");
  constexpr int TM = DUO_BM, TN = DUO_BN, NST = 3, LA = 2, LB = 4;     // LA, LB: 1 KB load instructions per wavefront and step
  constexpr int SA = TM * DUO_BK, SB = TN * DUO_BK;                    // elements of a stage
  __shared__ __attribute__((aligned(1024))) uint16_t smem[NST * (SA + SB)];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int group = p.per_slot || !p.class_order ? blockIdx.z : p.class_order[blockIdx.z];
  const int ntx = gridDim.x, nt = ntx * gridDim.y;
  int tile = blockIdx.y * ntx + blockIdx.x;
  const int R = nt % 256 == 0 ? 256 : nt % 128 == 0 ? 128 : nt % 64 == 0 ? 64 : 0;   // as in the large tile's kernel
  if (R) xcd_block(tile, ntx, R, tile);
  const int mt = tile / ntx, n0 = (tile - mt * ntx) * TN;
  const int row0 = mt * TM, row1 = min(p.M, row0 + TM);
  const int q0 = p.per_slot ? group : p.first_slot[group], q1 = p.per_slot ? group + 1 : p.first_slot[group + 1];
  const int kbeg = p.slot_offsets[q0], K = p.slot_offsets[q1] - kbeg;
  if (K == 0) {
    if (p.skip_empty) return;
    float* const Co = static_cast<float*>(p.C) + (long long)group * p.c_group_stride;
    const int col = n0 + lane * 4;
    if (col < p.N)
      for (int r = row0 + wave; r < row1; r += GT / 64) *reinterpret_cast<float4*>(Co + (long long)r * p.N + col) = make_float4(0.f, 0.f, 0.f, 0.f);
    return;
  }
  const int rows = row1 - row0, cols = p.N - n0;
  const int lda = MODE == WGRAD2 ? p.d : 2 * p.f, ldb = MODE == WGRAD2 ? p.f : p.d;
  const uint16_t* const a_base = static_cast<const uint16_t*>(p.A) + (long long)kbeg * lda + row0;
  const uint16_t* const b_base = static_cast<const uint16_t*>(p.B) + (long long)kbeg * ldb + n0;
  auto swizzle = [](int k) { return (k & 3) | (((k >> 3) & 1) << 2); };
  // byte offset of this lane's 16 bytes for instruction j of an operand (its immediate, j KB, taken back out) and their reduction
  // index in the step; columns beyond the operand's extent are clamped (they only reach outputs never stored), indices
  // beyond K read from outside the buffer: zeros
  unsigned vo[LA + LB];
  int kr[LA + LB];
#pragma unroll
  for (int j = 0; j < LA + LB; ++j) {
    const bool right = j >= LA;   // an instruction brings 2 indices of the right operand, 4 of the left one
    const int i = right ? j - LA : j, q = wave * (right ? LB : LA) + i, sh = right ? 5 : 4;
    kr[j] = (q << (6 - sh)) + (lane >> sh);
    const int c = (lane & ((1 << sh) - 1)) ^ (2 * swizzle(kr[j]));
    vo[j] = (unsigned)(kr[j] * (right ? ldb : lda) + (c * 8 < (right ? cols : rows) ? c * 8 : 0)) * 2u + 4096u - (unsigned)(i * 1024);
  }
  const unsigned ldsA = (unsigned)(size_t)SYMI_LPTR(smem) + wave * (LA * 1024);
  const unsigned ldsB = (unsigned)(size_t)SYMI_LPTR(smem + NST * SA) + wave * (LB * 1024);
  const int nk = (K + DUO_BK - 1) / DUO_BK;
  // a tile of at most 64 rows: the lower wavefronts have no outputs
  const bool idle = wave >= 2 && rows <= TM / 2;
  auto load_one = [&](auto jc, unsigned v, intx4 rsrc) {
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen offset:%2 lds" ::"v"(v), "s"(rsrc), "n"(decltype(jc)::value * 1024) : "memory");
  };
  auto load = [&](auto rightc, unsigned dst, const uint16_t* src, int left) {
    constexpr bool right = decltype(rightc)::value != 0;
    const unsigned long long a = (unsigned long long)src - 4096;
    const intx4 rsrc = {(int)(unsigned)a, (int)((unsigned)(a >> 32) & 0xffffu), (int)OUTSIDE, 0x00020000};
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" ::"s"(dst) : "memory");   // the wait state of an M0 write
    unroll<right ? LB : LA>([&](auto jc) {
      constexpr int x = (right ? LA : 0) + decltype(jc)::value;
      load_one(jc, kr[x] < left ? vo[x] : OUTSIDE, rsrc);
    });
  };
  auto issue = [&](int t, int st) {
    const int k0 = t * DUO_BK;
    load(IC<0>{}, ldsA + st * (SA * 2), a_base + (long long)k0 * lda, K - k0);
    load(IC<1>{}, ldsB + st * (SB * 2), b_base + (long long)k0 * ldb, K - k0);
  };
  const int g4 = lane >> 4, jj = lane & 15, tr = 8 * g4 + (jj >> 2);   // tr: k-row of a transposing read
  unsigned adA[4], adB[8];   // elements
#pragma unroll
  for (int i = 0; i < 4; ++i) adA[i] = tr * TM + (((wm * 4 + i) ^ swizzle(tr)) * 16) + (jj & 3) * 4;
#pragma unroll
  for (int j = 0; j < 8; ++j) adB[j] = NST * SA + tr * TN + (((wn * 8 + j) ^ swizzle(tr)) * 16) + (jj & 3) * 4;
  auto frag = [&](const uint16_t* q, int pitch) -> bf16x8 {
    union { shortx4 h[2]; bf16x8 v; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)SYMI_LPTR(q));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((shortx4 __attribute__((address_space(3)))*)SYMI_LPTR(q + 4 * pitch));
    return u.v;
  };
  floatx4 acc[4][8];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  issue(0, 0);
  issue(1, 1);
  int st = 0;
  for (int t = 0; t < nk; ++t) {
    // my loads of step t have landed (those of the next step may fly); behind the barrier everybody's, and the stage of step t - 1 is free
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0F70 + LA + LB);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(t + 2, st == 0 ? 2 : st - 1);
    if (!idle) {
      bf16x8 fa[4], fb[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) fa[i] = frag(smem + st * SA + adA[i], TM);
#pragma unroll
      for (int j = 0; j < 8; ++j) fb[j] = frag(smem + st * SB + adB[j], TN);
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    // my fragment reads of this step are through before its stage is filled again, behind the next barrier
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);
    st = st == NST - 1 ? 0 : st + 1;
  }
  wait_vmcnt0();
  __syncthreads();   // nobody's loads are in flight and nobody reads operands any more: the stages become the staging area
  if (idle) return;
  SavedUV<4> saved[2];   // write_tile's, of the hidden gradient alone
  write_tile<MODE, 2, 4>(p, smem + wave * (NST * (SA + SB) / 4), acc, row0, row1, group, n0, wm, wn, lane, -1, saved);
}

// ---------------------------------------------------------------- sum of reduction slices
// Runs behind FWD2 / BWD_DX (same stream): adds the partial tiles of every sliced tile in slice
// order and writes the bf16 rows of the product.  Workgroup = 16 rows of a tile, a lane four
// consecutive columns of four rows.  Returns at once if the product's tail was not sliced.
__global__ __launch_bounds__(256) void slice_sum_kernel(GemmParams p, int ntx) {
  const int tid = threadIdx.x;
  const int n_tiles = p.tile_map[0] * ntx;
  int full, sl;
  tail_slices(n_tiles, p.cus, p.K, full, sl);
  const int tile = full + blockIdx.y;
  if (sl < 2 || tile >= n_tiles) return;
  const int mt = tile / ntx;
  const int row0 = p.tile_map[4 + 4 * mt], row1 = p.tile_map[4 + 4 * mt + 1];
  const int n0 = (tile - mt * ntx) * BN;
  const float* part = p.partials + (size_t)blockIdx.y * sl * (BM * BN);
  const int c = (tid & 63) * 4;
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int r = blockIdx.x * 16 + it * 4 + (tid >> 6);
    const int row = row0 + r, col = n0 + c;
    if (row >= row1 || col >= p.N) continue;
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int z = 0; z < sl; ++z) {
      const float4 x = *reinterpret_cast<const float4*>(part + (size_t)z * (BM * BN) + r * BN + c);
      sum.x += x.x; sum.y += x.y; sum.z += x.z; sum.w += x.w;
    }
    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(p.C) + (long long)row * p.N + col) =
        make_uint2(pack_bf16x2(sum.x, sum.y), pack_bf16x2(sum.z, sum.w));
  }
}

// ---------------------------------------------------------------- fp32 products
// The same six products for fp32 activations and weights on the fp32 matrix instruction
// (32x32x2: 64 cycles for 4096 flops per SIMD, twice the rate of plain FMAs).  A wavefront
// computes 32-row x 32-column blocks; lane l holds row (left) or column (right) l % 32 of an
// operand, and of every 8 reduction indices the four 4*(l/32) .. +3: both operands agree on that
// order, so it only permutes the sum.  In the result, lane l holds column l % 32 and its 16
// registers the rows 8*(r/4) + 4*(l/32) + r%4: stores and the saved u, v are whole 128-byte lines.
// Two-level summation: every 16 reduction indices are summed in a fresh accumulator and then added,
// which keeps the rounding error of long reductions (weight gradients) near sqrt(K/16).
constexpr int F32_CHUNK = 16;

// What the fp32 kernels need to know about a product: its operands, their pitches and extents.
template <int MODE>
struct F32Operands {
  static constexpr bool VARM = MODE <= BWD_DX;
  static constexpr bool A_KC = VARM;                       // left operand reduction-contiguous
  static constexpr bool B_KC = MODE == FWD1 || MODE == FWD2;
  const float* A;    // first tile row (KC) or column 0 of the reduction's first row (KS)
  const float* B;
  long long lda, ldb;
  int row0, row1, group, K;

  // variable rows
  __device__ __forceinline__ void init_rows(const GemmParams& p, int r0, int r1, int slot) {
    row0 = r0;
    row1 = r1;
    group = slot;
    K = p.K;
    bind(p, 0);
  }
  // row tile y of the group that is z-th in the order of decreasing row counts, or group g itself
  __device__ __forceinline__ bool init(const GemmParams& p, int rows, int y, int z, int g = -1) {
    group = p.per_slot ? z : g >= 0 ? g : p.class_order[z];   // long reductions first
    row0 = y * rows;
    row1 = min(p.M, row0 + rows);
    const int q0 = p.per_slot ? group : p.first_slot[group], q1 = p.per_slot ? group + 1 : p.first_slot[group + 1];
    const int kbeg = p.slot_offsets[q0];
    K = p.slot_offsets[q1] - kbeg;
    if (K == 0 && p.skip_empty) return false;
    bind(p, kbeg);
    return true;
  }
  __device__ __forceinline__ void bind(const GemmParams& p, int kbeg) {
    lda = MODE == FWD2 ? p.f : (MODE == BWD_DX || MODE == WGRAD1) ? 2LL * p.f : p.d;
    ldb = (MODE == FWD1 || MODE == BWD_DX || MODE == WGRAD1) ? p.d : p.f;
    A = static_cast<const float*>(p.A) + (VARM ? (long long)row0 * lda : (long long)kbeg * lda + row0);
    B = static_cast<const float*>(p.B) + (VARM ? (long long)group * p.b_group_stride : (long long)kbeg * ldb);
  }
};

// value x (for FWD1 also its up half v) of output element (row, col)
template <int MODE>
__device__ __forceinline__ void f32_store(const GemmParams& p, int group, long long row, int col, float x, float v) {
  const long long f = p.f;
  if (MODE == FWD1) {
    float* UVo = static_cast<float*>(p.UVout);
    UVo[row * 2 * f + col] = x;
    UVo[row * 2 * f + f + col] = v;
    static_cast<float*>(p.H)[row * f + col] = silu_f(x) * v;
  } else if (MODE == FWD2 || MODE == BWD_DX) {
    static_cast<float*>(p.C)[row * p.N + col] = x;
  } else if (MODE == BWD_DH) {
    const float* UVi = static_cast<const float*>(p.UV);
    const float u = UVi[row * 2 * f + col], vv = UVi[row * 2 * f + f + col];
    const float sg = sigmoid_f(u);
    float* Co = static_cast<float*>(p.C);
    Co[row * 2 * f + col] = x * vv * sg * (1.f + u * (1.f - sg));
    Co[row * 2 * f + f + col] = x * u * sg;
  } else {
    (static_cast<float*>(p.C) + (long long)group * p.c_group_stride)[row * p.N + col] = x;
  }
}

// Tile of 64 rows x 128 columns (FWD1: the gate and up columns of 64 hidden units), four wavefronts of
// 32 x 64.  Tiles travel HBM -> LDS with direct-to-LDS loads, 32-deep steps in two stages: the next step's loads are in flight
// while the current one feeds the matrix pipes, one barrier per step.  Rows and columns beyond the tile's extent (N: the columns
// that exist) are clamped to a valid one (they only reach outputs that are never stored), reduction indices beyond K are zeros in both
// operands (offsets outside the buffer).  A wavefront whose outputs all lie outside multiplies nothing.
// LDS layouts, free of bank conflicts: reduction-contiguous [row][k], 16-byte chunk c of row r at c ^ ((r >> 1) & 7), read 16
// bytes per lane; reduction-strided [k][column] as loaded, chunk c of row k at c ^ (8 ((k >> 2) & 1)): the two
// halves of a wavefront read rows 4 apart, 32 banks apart.  With 128 columns a lane reads two neighbouring ones
// at a time, so block j of a wavefront holds its columns 2 l + j.
constexpr int F32_BM = 64;

template <int MODE>
__device__ __forceinline__ void f32_tile(const GemmParams& p, const F32Operands<MODE>& o, const int n0, const int N, float* const smem) {
  using Op = F32Operands<MODE>;
  constexpr int NBL = 2, KD = 32, F32_BN = 128;
  constexpr bool VARM = Op::VARM;
  constexpr bool PAIRS = !Op::B_KC;               // neighbouring columns in one lane
  constexpr int NST = 2;                          // stages
  constexpr int NLA = KD / 16, NLB = NLA * NBL;   // 1 KB load instructions per wavefront, operand and stage
  constexpr int SA = F32_BM * KD, SB = F32_BN * KD;   // elements of a stage
  float* const As = smem;
  float* const Bs = smem + NST * SA;
  const int K = o.K;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, r31 = lane & 31, hw = lane >> 5;

  auto swizzle = [](int r) { return (r >> 1) & 7; };   // of a [row][k] tile's chunks

  // byte offset of this lane's 16 bytes for instruction j of an operand (its immediate, j KB, taken back out) and their
  // reduction index in the step
  unsigned vo[NLA + NLB];
  int kr[NLA + NLB];
#pragma unroll
  for (int x = 0; x < NLA + NLB; ++x) {
    const bool right = x >= NLA;
    const int j = right ? x - NLA : x, q = wave * (right ? NLB : NLA) + j;
    const int ld = (int)(right ? o.ldb : o.lda), extent = right ? N - n0 : o.row1 - o.row0;
    unsigned e;
    if (right ? Op::B_KC : Op::A_KC) {   // 256 / KD rows
      const int r = q * (256 / KD) + lane / (KD / 4);
      kr[x] = ((lane & (KD / 4 - 1)) ^ swizzle(r)) * 4;
      // FWD1: the 64 tile columns of a wavefront are 32 gate and the 32 up columns of the same hidden units; a
      // wavefront loads either gate or up columns
      const int row = right && MODE == FWD1 ? (r >> 6) * 32 + (r & 31) : r;
      e = (unsigned)(min(row, extent - 1) * ld + kr[x]);
    } else {
      const int cpr = (right ? F32_BN : F32_BM) / 4;   // chunks of a row
      kr[x] = q * (64 / cpr) + lane / cpr;
      const int c = ((lane & (cpr - 1)) ^ (8 * ((kr[x] >> 2) & 1))) * 4;
      e = (unsigned)(kr[x] * ld + (c < extent ? c : 0));
    }
    vo[x] = e * 4u + 4096u - (unsigned)(j * 1024);
  }
  const float* const b0 = o.B + (Op::B_KC ? n0 * o.ldb : n0) + (MODE == FWD1 && (wave & 1) ? (long long)p.f * o.ldb : 0);
  const unsigned ldsA = (unsigned)(size_t)SYMI_LPTR(As) + wave * (NLA * 1024);
  const unsigned ldsB = (unsigned)(size_t)SYMI_LPTR(Bs) + wave * (NLB * 1024);
  auto load_one = [&](auto jc, unsigned v, intx4 rsrc) {
    asm volatile("buffer_load_dwordx4 %0, %1, 0 offen offset:%2 lds" ::"v"(v), "s"(rsrc), "n"(decltype(jc)::value * 1024) : "memory");
  };
  auto load = [&](auto rightc, unsigned dst, const float* src, int left, auto edge) {
    constexpr bool right = decltype(rightc)::value != 0;
    const unsigned long long a = (unsigned long long)src - 4096;
    const intx4 rsrc = {(int)(unsigned)a, (int)((unsigned)(a >> 32) & 0xffffu), (int)OUTSIDE, 0x00020000};
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" ::"s"(dst) : "memory");   // the wait state of an M0 write
    unroll<right ? NLB : NLA>([&](auto jc) {
      constexpr int x = (right ? NLA : 0) + decltype(jc)::value;
      load_one(jc, !decltype(edge)::value || kr[x] < left ? vo[x] : OUTSIDE, rsrc);
    });
  };
  auto issue = [&](int t, int st) {
    const int k0 = t * KD;
    const float* const sa = o.A + (Op::A_KC ? (long long)k0 : k0 * o.lda);
    const float* const sb = b0 + (Op::B_KC ? (long long)k0 : k0 * o.ldb);
    if (k0 + KD <= K) {
      load(IC<0>{}, ldsA + st * (SA * 4), sa, 0, std::false_type{});
      load(IC<1>{}, ldsB + st * (SB * 4), sb, 0, std::false_type{});
    } else {
      load(IC<0>{}, ldsA + st * (SA * 4), sa, K - k0, std::true_type{});
      load(IC<1>{}, ldsB + st * (SB * 4), sb, K - k0, std::true_type{});
    }
  };
  const int col0 = n0 + wn * (MODE == FWD1 ? 32 : 32 * NBL);
  const bool busy = wm * 32 < o.row1 - o.row0 && col0 < N;   // this wavefront holds outputs

  floatx16 acc[NBL];
#pragma unroll
  for (int j = 0; j < NBL; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  // element of As / Bs: KC chunk 2 s + hw of row, KS column of reduction index 4 hw (+ i + 8 s); the xor of a chunk
  const int kx = swizzle(r31);
  const int ra = Op::A_KC ? (wm * 32 + r31) * KD : hw * 4 * F32_BM + ((wm * 32 + r31) ^ (32 * hw));
  const int rb = Op::B_KC ? (wn * 32 * NBL + r31) * KD
                          : hw * 4 * F32_BN + ((wn * 32 * NBL + (PAIRS ? 2 : 1) * r31) ^ (32 * hw));
  auto multiply = [&](const float* const as, const float* const bs) {
#pragma unroll
    for (int c = 0; c < KD / F32_CHUNK; ++c) {
      floatx16 part[NBL];
#pragma unroll
      for (int j = 0; j < NBL; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) part[j][r] = 0.f;
#pragma unroll
      for (int s = 0; s < F32_CHUNK / 8; ++s) {
        const int k8 = c * F32_CHUNK + s * 8;   // reduction indices k8 + 4 hw + i
        float a[4], b[NBL][4];
        if (Op::A_KC) {
          const float4 q = *reinterpret_cast<const float4*>(as + ra + (((k8 / 4 + hw) ^ kx) * 4));
          a[0] = q.x; a[1] = q.y; a[2] = q.z; a[3] = q.w;
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) a[i] = as[ra + (k8 + i) * F32_BM];
        }
        if (PAIRS) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float2 q = *reinterpret_cast<const float2*>(bs + rb + (k8 + i) * F32_BN);
            b[0][i] = q.x; b[NBL - 1][i] = q.y;
          }
        } else {
#pragma unroll
          for (int j = 0; j < NBL; ++j) {
            if (Op::B_KC) {
              const float4 q = *reinterpret_cast<const float4*>(bs + rb + j * 32 * KD + (((k8 / 4 + hw) ^ kx) * 4));
              b[j][0] = q.x; b[j][1] = q.y; b[j][2] = q.z; b[j][3] = q.w;
            } else {
#pragma unroll
              for (int i = 0; i < 4; ++i) b[j][i] = bs[rb + (k8 + i) * F32_BN];
            }
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < NBL; ++j)
            part[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j][i], part[j], 0, 0, 0);
      }
#pragma unroll
      for (int j = 0; j < NBL; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] += part[j][r];
    }
  };
  const int nk = (K + KD - 1) / KD;
#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < nk) issue(t, t);
  int st = 0;
  for (int t = 0; t < nk; ++t) {
    // my loads of step t have landed and my reads of step t - 1 are through; behind the barrier everybody's, and its
    // stage may be filled
    __builtin_amdgcn_s_waitcnt(0x0070);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (t + NST - 1 < nk) issue(t + NST - 1, st == 0 ? NST - 1 : st - 1);
    if (busy) multiply(As + st * SA, Bs + st * SB);
    asm volatile("" ::: "memory");
    st = st == NST - 1 ? 0 : st + 1;
  }

  if (!busy) return;
  // Stores past the tile's end go outside the buffer; no branch keeps the loads of a whole block from flying together.
  constexpr int VW = PAIRS ? 2 : 1;   // neighbouring columns of a lane
  const long long rb0 = o.row0 + wm * 32;
  const int left = o.row1 - (int)rb0, twof = 2 * p.f;
  auto row_of = [&](int r) { return 8 * (r >> 2) + 4 * hw + (r & 3); };
  auto store = [&](float* base, bool in, unsigned at, float x, float y) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)OUTSIDE, 0x00020000);
    const int ofs = (int)(in ? at * 4u : OUTSIDE);
    if (VW == 2) __builtin_amdgcn_raw_buffer_store_b64(uintx2{__float_as_uint(x), __float_as_uint(y)}, rsrc, ofs, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), rsrc, ofs, 0, 0);
  };
#pragma unroll
  for (int j = 0; j < (MODE == FWD1 || PAIRS ? 1 : NBL); ++j) {
    const int col = col0 + j * 32 + VW * r31;
    const bool in_col = col < N;   // N is even
    if constexpr (MODE == FWD1) {
      float* const UVo = static_cast<float*>(p.UVout) + rb0 * twof;
      float* const Ho = static_cast<float*>(p.H) + rb0 * p.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool in = in_col && row_of(r) < left;
        const float u = acc[0][r], v = acc[NBL - 1][r];
        const unsigned at = (unsigned)(row_of(r) * twof + col);
        store(UVo, in, at, u, 0.f);
        store(UVo + p.f, in, at, v, 0.f);
        store(Ho, in, (unsigned)(row_of(r) * p.f + col), silu_f(u) * v, 0.f);
      }
    } else if constexpr (MODE == BWD_DH) {
      const float* const UVi = static_cast<const float*>(p.UV) + rb0 * twof + min(col, N - VW);
      float* const Co = static_cast<float*>(p.C) + rb0 * twof;
      float u[16][VW], v[16][VW];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float* const q = UVi + (long long)min(row_of(r), left - 1) * twof;
#pragma unroll
        for (int x = 0; x < VW; ++x) {
          u[r][x] = q[x];
          v[r][x] = q[p.f + x];
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float du[2] = {0.f, 0.f}, dv[2] = {0.f, 0.f};
#pragma unroll
        for (int x = 0; x < VW; ++x) {
          const float dh = acc[j + x][r], sg = sigmoid_f(u[r][x]);
          du[x] = dh * v[r][x] * sg * (1.f + u[r][x] * (1.f - sg));
          dv[x] = dh * u[r][x] * sg;
        }
        const bool in = in_col && row_of(r) < left;
        const unsigned at = (unsigned)(row_of(r) * twof + col);
        store(Co, in, at, du[0], du[1]);
        store(Co + p.f, in, at, dv[0], dv[1]);
      }
    } else {
      float* const Co = static_cast<float*>(p.C) + (VARM ? 0 : (long long)o.group * p.c_group_stride) + rb0 * p.N;
#pragma unroll
      for (int r = 0; r < 16; ++r)
        store(Co, in_col && row_of(r) < left, (unsigned)(row_of(r) * p.N + col), acc[j][r], acc[NBL - 1][r]);
    }
  }
}

// The weight gradients of groups with a few rows each, whose time is that of the stores: one tile per workgroup.
template <int MODE>
__global__ __launch_bounds__(256, 3) void gemm_f32_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(1024))) float smem[2 * (F32_BM + 128) * 32];
  F32Operands<MODE> o;
  if (!o.init(p, F32_BM, blockIdx.y, blockIdx.z)) return;
  f32_tile<MODE>(p, o, blockIdx.x * 128, p.N, smem);
}

// ---------------------------------------------------------------- fp32 products on the bf16 matrix instruction
// An fp32 value is the sum of three bf16 values to 24 bits: x = x0 + x1 + x2, each the bf16 nearest to what the ones
// before leave.  A product then is x0 y0 + (x0 y1 + x1 y0) + (x1 y1 + x0 y2 + x2 y0) and terms of up to 2^-24.2 of it (2^-27.5 rms): six matrix
// instructions at 16 times the rate of the fp32 one.  A step of 32 indices is summed from zero, the small terms first, and
// then added to the total, half as many additions as of 16 products each on the fp32 instruction: error against
// binary64 (relative 2-norm) Y 2.4e-7 -> 1.9e-7, dX 2.8e-7 -> 2.2e-7, dW1 2.7e-7 -> 2.1e-7 on 24 classes of d = 328, f = 872,
// 8997 rows.  Every value is taken 2^24 times as large (the sum goes back by 2^-48), so that the third part of the smallest
// fp32 number is a normal bf16 number and no part is lost, whatever stands beside it (16 multiplications per thread and step, backward
// of the shape above up to 1 % longer; unscaled, values up to 2^-134 had no parts at all).  What leaves the range for it, infinities, NaN,
// values from 2^104 and sums from 2^80 on, leaves a sum that is not finite, and the tile is computed once more on the fp32
// instruction (f32_tile).  Weight gradients of a class (or slot) with one or two rows are computed there alone: the terms left
// out are more than the few additions save.  Relative 2-norm, 1e-8, fp32 instruction : split, 1 row 2.5 : 3.5 (largest 6.0 : 14.2), 2 rows 3.2 :
// 3.4, 3 rows 3.6 : 3.4, 8 rows 5.3 : 3.5, 128 rows 9.2 : 6.0; backward of 24 classes of d = 328, f = 872, twelve with one row and twelve with 600,
// 296 -> 304 us.
// What that costs, 24 classes of 375 rows, no infinity / one / one in every 64 rows: forward 179 / 193 / 406 us, backward 344 / 361 / 859.  A
// tile's values alone decide it, so a row's bits depend on the up to 63 rows beside it where one of them is out of the range.
// Tile of 64 x 64 (FWD1: 32 hidden units), four wavefronts of 32 x 32, three workgroups per compute unit that stay and
// take one tile after the other.  A thread loads 16 values of a step into registers, two to three steps ahead, splits
// them beside the matrix instructions of the step before and writes the planes to the other of two LDS stages; one barrier per step.
// Bound by the vector instructions of the splits next to the matrix instructions (28 % of the matrix pipes' time is theirs
// with 128 x 128 tiles), and where the tiles are few by the last round of them.  Step of the shape above 767 -> 598 - 606 us, forward of
// 24 classes of d = 256, f = 576, 18096 rows 154 -> 118, backward of 4 classes of d = 104, f = 896, 1412 rows 107 -> 78; 75 drawn
// layers 1.10 (0.96 - 1.41).  Tried and dropped: 128 x 128 tiles with eight wavefronts (that step 620: fewer splits per product, but 273
// tiles of the input gradient are two rounds of 256), half of the wavefronts loading and splitting for the other half (616 - 640), everything
// in each wavefront between two barriers (626 - 667), planes by truncation (2.4e-7 -> 3.1e-7).
// LDS layouts, free of bank conflicts: reduction-contiguous [row][32 k], 16-byte chunk c of row r at c ^ s with s = 0, 2, 3, 1
// for (r >> 2) & 3; reduction-strided [k][64 columns] as loaded, 32-byte piece c of row k at c ^ (((k >> 1) & 1) + 2 ((k >> 3) & 1)), read transposing.
constexpr int F32S_T = 64, F32S_BK = 32;   // tile edge, step
constexpr float F32S_SCALE = 0x1p24f, F32S_BACK = 0x1p-48f;
constexpr int F32S_FEW = 2;                // rows of a class up to which its gradients are the fp32 instruction's
constexpr int F32S_FLAGS = 1024;           // words of flags: for 32768 tiles of a workgroup, some 400 GB of outputs

// The tiles of a product that one workgroup computes, one after the other.  XCD x (workgroup number mod 8) takes an eighth of
// the row tiles with all their columns, or of every class's tiles, the classes in order of decreasing row count.
struct F32Tile { int row0, row1, group, bx, kbeg, K; };

__device__ __forceinline__ int const_i32(const int32_t* q) {   // a scalar load: written by an earlier kernel
  return *(const int32_t __attribute__((address_space(4)))*)(unsigned long long)q;
}

template <int MODE>
struct F32Walk {
  static constexpr int T = F32S_T;
  static constexpr bool VARM = MODE <= BWD_DX;
  const GemmParams& p;
  int groups, x, s, cx, ntx, lo, n, per, nt, i;
  __device__ __forceinline__ F32Walk(const GemmParams& p_, int groups_) : p(p_), groups(groups_) {
    const int G = gridDim.x, b = blockIdx.x;
    x = b & 7;
    s = b >> 3;
    cx = (G - x + 7) >> 3;
    i = 0;
    if (VARM) {
      ntx = (p.N + (MODE == FWD1 ? T / 2 : T) - 1) / (MODE == FWD1 ? T / 2 : T);
      const long long all = (long long)const_i32(p.tile_map) * ntx;
      lo = (int)(all * x / 8);
      n = (int)(all * (x + 1) / 8) - lo;
    } else {
      ntx = (p.N + T - 1) / T;
      nt = ntx * ((p.M + T - 1) / T);
      per = (nt + 7) / 8;
      n = groups * per;
    }
  }
  __device__ __forceinline__ bool next(F32Tile& t) {
    for (;; ++i) {
      if (i * cx >= n) return false;
      const int u = i * cx + (!VARM && (i & 1) ? cx - 1 - s : s);   // the larger classes come first: there and back
      if (u >= n) continue;
      if (VARM) {
        const int mt = (lo + u) / ntx;
        const int entry = const_i32(p.tile_map + 4 + 2 * mt + 1);
        t.bx = lo + u - mt * ntx;
        t.row0 = const_i32(p.tile_map + 4 + 2 * mt);
        t.row1 = t.row0 + (entry >> 16) + 1;
        t.group = entry & 0xffff;
        t.kbeg = 0;
        t.K = p.K;
      } else {
        const int c = u / per, at = ((x + c) & 7) * per + u - c * per;
        if (at >= nt) continue;
        const int mt = at / ntx;
        t.bx = at - mt * ntx;
        t.row0 = mt * T;
        t.row1 = min(p.M, t.row0 + T);
        t.group = p.per_slot ? c : const_i32(p.class_order + c);
        const int q0 = p.per_slot ? c : const_i32(p.first_slot + t.group), q1 = p.per_slot ? c + 1 : const_i32(p.first_slot + t.group + 1);
        t.kbeg = const_i32(p.slot_offsets + q0);
        t.K = const_i32(p.slot_offsets + q1) - t.kbeg;
      }
      ++i;
      return true;
    }
  }
};

template <int MODE>
__global__ __launch_bounds__(256, 3) void gemm_f32_split_kernel(GemmParams p, int groups) {
  using Op = F32Operands<MODE>;
  constexpr int T = F32S_T;
  constexpr bool VARM = Op::VARM;
  constexpr int MI = 2, NJ = 2, WR = 32, WC = 32;            // 16 x 16 blocks, rows and columns of a wavefront
  constexpr int PL = T * F32S_BK * 2, ST = 6 * PL;           // bytes: a plane, a stage
  constexpr int EXACT = 2 * 4 * (F32_BM + 128) * 32;
  __shared__ __attribute__((aligned(1024))) char smem[2 * ST > EXACT ? 2 * ST : EXACT];
  __shared__ unsigned redo[F32S_FLAGS + 1];   // tiles for the fp32 instruction; any at all
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, g4 = lane >> 4, jj = lane & 15;
  const int N = MODE == FWD1 ? p.f : p.N;
  const int lda = MODE == FWD2 ? p.f : (MODE == BWD_DX || MODE == WGRAD1) ? 2 * p.f : p.d;
  const int ldb = (MODE == FWD1 || MODE == BWD_DX || MODE == WGRAD1) ? p.d : p.f;
  auto swizzle = [](int k) { return ((k >> 1) & 1) | (((k >> 3) & 1) << 1); };
  auto kc_swz = [](int r) { const int a = (r >> 2) & 3; return ((a ^ (a >> 1)) & 1) << 1 | (a >> 1); };
  auto meet = [] {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  for (int q = tid; q <= F32S_FLAGS; q += 256) redo[q] = 0;
  meet();   // a tile without a split sum is flagged at once
  auto summed = [](const F32Tile& tile) { return VARM || tile.K > F32S_FEW; };

  // ---- loads: two of the left operand, two of the right one per thread and step
  unsigned ls[4], vo[4];   // byte offsets inside a stage and in memory
  int kr[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const int q = tid + 256 * (x & 1);
    if (x < 2 ? Op::A_KC : Op::B_KC) {
      const int r = q >> 3;
      kr[x] = (q & 7) * 4;
      ls[x] = r * 64 + (((kr[x] >> 3) ^ kc_swz(r)) << 4) + ((kr[x] >> 2) & 1) * 8;
    } else {
      kr[x] = q / (T / 4);
      ls[x] = kr[x] * (2 * T) + ((8 * (q & (T / 4 - 1))) ^ (swizzle(kr[x]) << 5));
    }
    if (x >= 2) ls[x] += 3 * PL;
    vo[x] = 0;
  }
  F32Walk<MODE> ahead(p, groups);
  F32Tile nx;
  bool more = ahead.next(nx);
  const float* a0 = nullptr;
  const float* b0 = nullptr;
  int lK = 0, lk = 0;
  __amdgpu_buffer_rsrc_t ra, rb;
  int left = 0;
  auto buf = [](const float* q) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(q), 0, (int)OUTSIDE, 0x00020000); };
  auto next_step = [&] {   // where the next step's loads are; zeros beyond the last one
    while (lk >= lK && more) {
      const F32Tile t = nx;
      more = ahead.next(nx);
      lK = summed(t) ? t.K : 0;
      lk = 0;
      const int n0 = t.bx * (MODE == FWD1 ? T / 2 : T);
      a0 = static_cast<const float*>(p.A) + (VARM ? (long long)t.row0 * lda : (long long)t.kbeg * lda + t.row0);
      b0 = static_cast<const float*>(p.B) + (VARM ? (long long)t.group * p.b_group_stride : (long long)t.kbeg * ldb) + (Op::B_KC ? (long long)n0 * ldb : n0);
      if (MODE == FWD1 && (wave & 2)) b0 += (long long)p.f * ldb;   // a wavefront loads gate or up columns
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int q = tid + 256 * (x & 1), extent = x < 2 ? t.row1 - t.row0 : N - n0, ld = x < 2 ? lda : ldb;
        if (x < 2 ? Op::A_KC : Op::B_KC) {
          const int r = q >> 3;   // FWD1: every 32 columns are 16 gate and the 16 up columns of the same hidden units
          vo[x] = 4u * (unsigned)(min(x >= 2 && MODE == FWD1 ? (r >> 5) * 16 + (r & 15) : r, extent - 1) * ld + kr[x]);
        } else {
          const int c = (q & (T / 4 - 1)) * 4;
          vo[x] = 4u * (unsigned)(kr[x] * ld + (c < extent ? c : 0));
        }
      }
    }
    left = lK - lk;
    ra = buf(a0 + (Op::A_KC ? (long long)lk : (long long)lk * lda));
    rb = buf(b0 + (Op::B_KC ? (long long)lk : (long long)lk * ldb));
    if (left > 0) lk += F32S_BK;
  };
  uintx4 sg[2][4];
  auto load = [&](auto sc, auto xc) {
    constexpr int x = decltype(xc)::value;
    sg[decltype(sc)::value][x] = __builtin_amdgcn_raw_buffer_load_b128(x < 2 ? ra : rb, (int)(kr[x] < left ? vo[x] : OUTSIDE), 0, 0);
  };
  // plane q of load x: the bf16 nearest to what is left of the value
  auto split = [&](auto sc, auto xc, auto qc) {
    constexpr int S = decltype(sc)::value, x = decltype(xc)::value, q = decltype(qc)::value;
    uintx4& v = sg[S][x];
    if constexpr (q == 0) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(__uint_as_float(v[e]) * F32S_SCALE);
    }
    const unsigned lo = pack_bf16x2(__uint_as_float(v[0]), __uint_as_float(v[1])), hi = pack_bf16x2(__uint_as_float(v[2]), __uint_as_float(v[3]));
    *reinterpret_cast<uint2*>(smem + S * ST + ls[x] + q * PL) = make_uint2(lo, hi);
    if constexpr (q < 2) {
      v[0] = __float_as_uint(__uint_as_float(v[0]) - __uint_as_float(lo << 16));
      v[1] = __float_as_uint(__uint_as_float(v[1]) - __uint_as_float(lo & 0xffff0000u));
      v[2] = __float_as_uint(__uint_as_float(v[2]) - __uint_as_float(hi << 16));
      v[3] = __float_as_uint(__uint_as_float(v[3]) - __uint_as_float(hi & 0xffff0000u));
    }
  };

  // ---- fragments
  unsigned adA[Op::A_KC ? 1 : MI], adB[Op::B_KC ? 1 : NJ];   // byte addresses of a lane's fragments in stage 0
  const unsigned lds = (unsigned)(size_t)SYMI_LPTR(smem);
  {
    const unsigned kc = jj * 64 + ((g4 ^ kc_swz(jj)) << 4), ks = (8 * g4 + (jj >> 2)) * 2 * T + (jj & 3) * 8;
    const int sw = swizzle(8 * g4 + (jj >> 2));
#pragma unroll
    for (int i = 0; i < (Op::A_KC ? 1 : MI); ++i) adA[i] = lds + (Op::A_KC ? wm * WR * 64 + kc : ks + (((wm * MI + i) ^ sw) << 5));
#pragma unroll
    for (int j = 0; j < (Op::B_KC ? 1 : NJ); ++j) adB[j] = lds + 3 * PL + (Op::B_KC ? wn * WC * 64 + kc : ks + (((wn * NJ + j) ^ sw) << 5));
  }
  // Reads and matrix instructions are inline assembly in the order in which they are to be issued: left to itself the compiler
  // reads a fragment just ahead of its use and waits for it.
  bf16x8 fa[3][MI], fb[4][NJ];   // fb[0], fb[3]: plane 0 of even and odd steps
  auto read = [&](bf16x8& f, auto kcc, auto ofsc, unsigned at) {
    constexpr int OFS = decltype(ofsc)::value;
    if constexpr (decltype(kcc)::value) {
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f) : "v"(at), "n"(OFS));
    } else {
      shortx4 x, y;
      asm volatile("ds_read_b64_tr_b16 %0, %2 offset:%3\n\tds_read_b64_tr_b16 %1, %2 offset:%4"
                   : "=&v"(x), "=&v"(y) : "v"(at), "n"(OFS), "n"(OFS + 8 * T));
      union { shortx4 h[2]; bf16x8 v; } u;
      u.h[0] = x;
      u.h[1] = y;
      f = u.v;
    }
  };
  // fragment r of planes qa, qb (qb into register set fb[sb]) of stage S: the left operand's first
  auto read_frag = [&](auto sc, auto qac, auto qbc, auto sbc, auto rc) {
    constexpr int S = decltype(sc)::value, QA = decltype(qac)::value, QB = decltype(qbc)::value, SB = decltype(sbc)::value, r = decltype(rc)::value;
    if constexpr (r < MI) read(fa[QA][r], std::integral_constant<bool, Op::A_KC>{}, IC<S * ST + QA * PL + (Op::A_KC ? r * 1024 : 0)>{}, adA[Op::A_KC ? 0 : r]);
    else if constexpr (r < MI + NJ)
      read(fb[SB][r - MI], std::integral_constant<bool, Op::B_KC>{}, IC<S * ST + QB * PL + (Op::B_KC ? (r - MI) * 1024 : 0)>{}, adB[Op::B_KC ? 0 : r - MI]);
  };
  auto landed = [] { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };
  floatx4 acc[MI][NJ], c[MI][NJ];
  auto add = [](floatx4& to, const floatx4& x) {
#pragma unroll
    for (int e = 0; e < 4; ++e) to[e] = fmaf(x[e], F32S_BACK, to[e]);
  };
  constexpr int NP = MI * NJ, PS = 5 * NP / 12;
  static_assert(MI + NJ <= NP && 12 * PS <= 5 * NP, "a phase has room for its reads, a step for its splits");
  // One step, stage S: six phases, each the product of two planes, the small ones first.  Beside them go the reads of the
  // next phases' fragments, and in the first three the next step's splits into the other stage with the loads of the step
  // after the next but one; in the last one the other stage is entered.
  auto phase = [&](auto sc, auto pc, auto qac, auto qbc) {
    constexpr int S = decltype(sc)::value, P = decltype(pc)::value, QA = decltype(qac)::value, QB = decltype(qbc)::value;
    __builtin_amdgcn_sched_barrier(0);
    unroll<NP>([&](auto mc) {
      constexpr int m = decltype(mc)::value, i = m / NJ, j = m % NJ;
      if constexpr (P == 0) {
        asm volatile("" : "+v"(c[i][j]));
        add(acc[i][j], c[i][j]);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=&v"(c[i][j]) : "v"(fb[QB][j]), "v"(fa[QA][i]));
      } else {
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c[i][j]) : "v"(fb[QB][j]), "v"(fa[QA][i]));
      }
      if constexpr (P == 0) read_frag(sc, IC<0>{}, IC<2>{}, IC<2>{}, mc);
      if constexpr (P == 1) read_frag(sc, IC<1>{}, IC<1>{}, IC<1>{}, mc);
      if constexpr (P == 5) read_frag(IC<S ^ 1>{}, IC<2>{}, IC<0>{}, IC<S ? 0 : 3>{}, mc);
      constexpr int n = P * NP + m, piece = n / PS;
      if constexpr (n % PS == 0 && piece < 12) {
        constexpr int x = piece / 3, q = piece % 3;
        split(IC<S ^ 1>{}, IC<x>{}, IC<q>{});
        if constexpr (q == 2) load(IC<S ^ 1>{}, IC<x>{});
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto step = [&](auto sc) {
    constexpr int S = decltype(sc)::value;
    next_step();
    landed();
    phase(sc, IC<0>{}, IC<2>{}, IC<S ? 3 : 0>{});
    landed();
    phase(sc, IC<1>{}, IC<0>{}, IC<2>{});
    landed();
    phase(sc, IC<2>{}, IC<1>{}, IC<1>{});
    phase(sc, IC<3>{}, IC<1>{}, IC<S ? 3 : 0>{});
    phase(sc, IC<4>{}, IC<0>{}, IC<1>{});
    meet();
    phase(sc, IC<5>{}, IC<0>{}, IC<S ? 3 : 0>{});
  };

  F32Walk<MODE> walk(p, groups);
  F32Tile t;
  bool have = walk.next(t);
  int tiles = 0, k0 = 0;
  auto clear = [&] {
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = c[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  };
  auto write_out = [&] {
    bool bad = !summed(t) && t.K > 0;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) bad |= !(fabsf(acc[i][j][e]) <= 3.4e38f);
    if (bad) {
      atomicOr(&redo[(tiles >> 5) & (F32S_FLAGS - 1)], 1u << (tiles & 31));
      redo[F32S_FLAGS] = 1;
    }
    if (!summed(t) && (t.K > 0 || p.skip_empty)) return;
    const int n0 = t.bx * (MODE == FWD1 ? T / 2 : T);
    const long long rb0 = t.row0 + wm * WR;
    const int rows = t.row1 - (int)rb0, twof = 2 * p.f;
    auto store = [&](float* base, bool in, unsigned at, floatx4 x) {
      const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)OUTSIDE, 0x00020000);
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, x), rsrc, (int)(in ? at * 4u : OUTSIDE), 0, 0);
    };
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int row = 16 * i + jj;
      if constexpr (MODE == FWD1) {
        float* const UVo = static_cast<float*>(p.UVout) + rb0 * twof;
        float* const Ho = static_cast<float*>(p.H) + rb0 * p.f;
        const int col = n0 + wn * 16 + 4 * g4;
        const bool in = row < rows && col < N;
        floatx4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = silu_f(acc[i][0][e]) * acc[i][1][e];
        store(UVo, in, (unsigned)(row * twof + col), acc[i][0]);
        store(UVo + p.f, in, (unsigned)(row * twof + col), acc[i][1]);
        store(Ho, in, (unsigned)(row * p.f + col), h);
      } else if constexpr (MODE == BWD_DH) {
        float* const Co = static_cast<float*>(p.C) + rb0 * twof;
        floatx4 u[NJ], v[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const float* const q = static_cast<const float*>(p.UV) + (rb0 + min(row, rows - 1)) * twof + min(n0 + wn * WC + 16 * j + 4 * g4, N - 4);
          u[j] = *reinterpret_cast<const floatx4*>(q);
          v[j] = *reinterpret_cast<const floatx4*>(q + p.f);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int col = n0 + wn * WC + 16 * j + 4 * g4;
          const bool in = row < rows && col < N;
          floatx4 du, dv;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float dh = acc[i][j][e], u_ = u[j][e], sgm = sigmoid_f(u_);
            du[e] = dh * v[j][e] * sgm * (1.f + u_ * (1.f - sgm));
            dv[e] = dh * u_ * sgm;
          }
          store(Co, in, (unsigned)(row * twof + col), du);
          store(Co + p.f, in, (unsigned)(row * twof + col), dv);
        }
      } else {
        float* const Co = static_cast<float*>(p.C) + (VARM ? 0 : (long long)t.group * p.c_group_stride) + rb0 * p.N;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int col = n0 + wn * WC + 16 * j + 4 * g4;
          store(Co, row < rows && col < N, (unsigned)(row * p.N + col), acc[i][j]);
        }
      }
    }
  };
  auto advance = [&] {   // the next tile with a sum
    do {
      write_out();
      ++tiles;
      have = walk.next(t);
      clear();
    } while (have && !summed(t));
    k0 = 0;
  };
  auto last_step = [&]() -> bool {   // behind a step: the tile's sums are complete
    k0 += F32S_BK;
    if (k0 < t.K) return false;
    // the next step's fragments are kept until they have landed
    landed();
#pragma unroll
    for (int i = 0; i < MI; ++i) asm volatile("" : "+v"(fa[2][i]));
#pragma unroll
    for (int j = 0; j < NJ; ++j) asm volatile("" : "+v"(fb[0][j]), "+v"(fb[3][j]));
    asm volatile("s_nop 15" ::: "memory");   // the last matrix instruction's results
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        asm volatile("" : "+v"(c[i][j]));
        add(acc[i][j], c[i][j]);
      }
    advance();
    return !have;
  };
  clear();
#pragma unroll
  for (int j = 0; j < NJ; ++j) fb[0][j] = fb[3][j] = bf16x8{};
  while (have && !summed(t)) {
    write_out();
    ++tiles;
    have = walk.next(t);
  }
  if (have) {
    next_step();
    unroll<4>([&](auto x) { load(IC<0>{}, x); });
    __builtin_amdgcn_sched_barrier(0);
    next_step();
    unroll<4>([&](auto x) { load(IC<1>{}, x); });
    __builtin_amdgcn_sched_barrier(0);
    next_step();
    unroll<4>([&](auto x) {
      split(IC<0>{}, x, IC<0>{});
      split(IC<0>{}, x, IC<1>{});
      split(IC<0>{}, x, IC<2>{});
      load(IC<0>{}, x);
    });
    meet();
    unroll<MI + NJ>([&](auto r) { read_frag(IC<0>{}, IC<2>{}, IC<0>{}, IC<0>{}, r); });
    // with a break behind each step the compiler moved a dozen (weight gradients 44) scalars through vector registers in every second one
    for (bool on = true; on;) {
      step(IC<0>{});
      on = !last_step();
      if (on) {
        step(IC<1>{});
        on = !last_step();
      }
    }
  }

  // ---- tiles with a sum that is not finite, and those without a split sum: on the fp32 instruction
  meet();
  if (__builtin_amdgcn_readfirstlane(redo[F32S_FLAGS]) == 0) return;
  walk.i = 0;
  for (int n = 0; walk.next(t); ++n) {
    // a tile without rows has no flag; should tiles share their flags, it may not be written all the same (skip_empty)
    if (t.K == 0 || !(__builtin_amdgcn_readfirstlane(redo[(n >> 5) & (F32S_FLAGS - 1)]) >> (n & 31) & 1)) continue;
    F32Operands<MODE> o;
    o.K = t.K;
    o.group = t.group;
    o.row0 = t.row0;
    o.row1 = t.row1;
    o.bind(p, t.kbeg);
    const int n0 = t.bx * (MODE == FWD1 ? T / 2 : T);
    meet();
    f32_tile<MODE>(p, o, n0, min(N, n0 + (MODE == FWD1 ? T / 2 : T)), reinterpret_cast<float*>(smem));
  }
}

// A small batch has too few 64 x 128 tiles to fill the chip, and the time of one tile is its
// reduction's latency.  Here a tile is 32 x 32 (FWD1: 32 hidden units, gate and up) and NW
// wavefronts share its reduction, each with its own range of reduction indices: 16-deep steps through an LDS ring of
// its own (direct-to-LDS loads, one to two steps ahead, no barrier); the sums meet in LDS in a fixed order.  A workgroup finds its
// rows from the slot offsets, about a microsecond, where a table was a launch of four; in the backward dh goes with dW2 and dX with dW1 in
// one launch, since neither fills the chip: c1's step 97 -> 85 us, 8 classes of d = 64, f = 864, 848 rows, backward 66 -> 47, 16 of
// d = 208, f = 464, 594 rows, forward 90 -> 48.
// Rows of a step are 64-byte segments, columns 128-byte ones; straight from memory into registers a load took 16 bytes
// of each of 32 rows, four loads to a cache line, and only one step flew: 512 rows in 8 slots of d = 512, f = 1280, the six
// products 53, 51, 32, 97, 20, 28 us -> 33, 26, 25, 48, 18, 24; 2048 rows in 16 slots of d = 128, f = 256 15, 11, 13, 16, 11,
// 13 -> 14, 9, 10, 13, 10, 11 (events around the launch).  Bound by latency: a table entry, the first loads, K / (16 NW) steps,
// the sum.
// Ring layouts, free of bank conflicts: reduction-contiguous [32 rows][16 k], 16-byte chunk c of row r at c ^ ((r >> 2) & 3);
// reduction-strided [16 k][32 columns], index k in row k ^ ((k >> 2) & 1): the two halves of a wavefront read indices 4 apart.
// NW wavefronts share a reduction, SUBS tiles in a workgroup.
template <int MODE, int NW, int SUBS>
struct F32Small {
  static constexpr int NT = 64 * NW * SUBS, NB = MODE == FWD1 ? 2 : 1;
  // stages: three workgroups of 48 KB per unit (FWD1, with two right operands, in two stages: c1's step 84.5 -> 83.1 us, forward of 24 classes of
  // d = 456, f = 224, 769 rows 46.4 -> 44.5), or two of 64 KB
  static constexpr int NST = NT == 256 && NB == 1 ? 3 : 2;
  static constexpr int SO = 32 * F32_CHUNK, RING = NST * (1 + NB) * SO;   // elements: an operand's step, a wavefront's ring
  static constexpr int LDS = NW * SUBS * RING;
};

// Row tile mt of the slots in order, TM rows each, counted from the slot offsets by all NT threads of the workgroup; SUBS
// groups of threads look for one each (sub: this thread's).  `found`: NT / 64 + 3 SUBS words.
template <int TM, int NT, int SUBS>
__device__ __forceinline__ bool find_rows(const int32_t* __restrict__ offs, int n_slots, int32_t* const found, const int (&mt)[SUBS],
                                          int sub, int& row0, int& row1, int& slot) {
  constexpr int NW = NT / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (n_slots + NT - 1) / NT, q0 = min(tid * per, n_slots), q1 = min(q0 + per, n_slots);
  int mine = 0;
  for (int q = q0; q < q1; ++q) mine += (offs[q + 1] - offs[q] + TM - 1) / TM;
  int incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) found[wave] = incl;
  __syncthreads();
  int n_tiles = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w < wave) incl += found[w];
    n_tiles += found[w];
  }
#pragma unroll
  for (int k = 0; k < SUBS; ++k) {
    if (mt[k] < incl && mt[k] >= incl - mine) {
      int i = mt[k] - (incl - mine), q = q0;
      for (;; ++q) {
        const int n = (offs[q + 1] - offs[q] + TM - 1) / TM;
        if (i < n) break;
        i -= n;
      }
      found[NW + 3 * k] = q;
      found[NW + 3 * k + 1] = offs[q] + i * TM;
      found[NW + 3 * k + 2] = min(offs[q] + i * TM + TM, offs[q + 1]);
    }
  }
  __syncthreads();
  const bool any = mt[sub] < n_tiles;
  slot = __builtin_amdgcn_readfirstlane(found[NW + 3 * sub]);
  row0 = __builtin_amdgcn_readfirstlane(found[NW + 3 * sub + 1]);
  row1 = __builtin_amdgcn_readfirstlane(found[NW + 3 * sub + 2]);
  __syncthreads();   // the words become part of the rings
  return any;
}

// The tiles of workgroup b of a product.  Rows are found from the slot offsets (no table is written where all
// products of a call are small), the classes are in no order.
template <int MODE, int NW, int SUBS>
__device__ __forceinline__ void f32_small_tile(const GemmParams& p, const int b, float* smem) {
  using Op = F32Operands<MODE>;
  using Sm = F32Small<MODE, NW, SUBS>;
  constexpr int NB = Sm::NB, NST = Sm::NST, SO = Sm::SO, RING = Sm::RING;
  constexpr int LDR = 40;                      // rows 4 apart are 32 banks apart
  static_assert(RING >= NB * 32 * LDR, "the sums reuse the ring");
  const int ntx = ((MODE == FWD1 ? p.f : p.N) + 31) / 32;
  const int sub = SUBS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * NW));
  Op o;
  int bx;
  bool any = true;   // a workgroup's last tile may not exist; its wavefronts meet the others all the same
  if constexpr (Op::VARM) {
    int mt[SUBS];
#pragma unroll
    for (int k = 0; k < SUBS; ++k) mt[k] = (b * SUBS + k) / ntx;
    bx = (b * SUBS + sub) % ntx;
    int row0, row1, slot;
    any = find_rows<32, Sm::NT, SUBS>(p.slot_offsets, p.n_slots, reinterpret_cast<int32_t*>(smem), mt, sub, row0, row1, slot);
    if (SUBS == 1 && !any) return;
    if (any) o.init_rows(p, row0, row1, slot);
  } else {
    static_assert(SUBS == 1, "one weight gradient tile in a workgroup");
    const int per = ntx * ((p.M + 31) / 32), z = b / per, at = b - z * per;
    bx = at % ntx;
    if (!o.init(p, 32, at / ntx, z, z)) return;
  }
  if (SUBS > 1 && !any) {
    __syncthreads();   // where the sums meet
    return;
  }
  smem += sub * NW * RING;
  const int K = o.K, N = MODE == FWD1 ? p.f : p.N;
  const int n0 = bx * 32;
  const int tid = threadIdx.x - sub * 64 * NW, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r31 = lane & 31, hw = lane >> 5;
  const int per = (K + NW * F32_CHUNK - 1) / (NW * F32_CHUNK) * F32_CHUNK;
  const int kbeg = wave * per, kend = min(K, kbeg + per);
  float* const ring = smem + wave * RING;

  // byte offset of this lane's 16 bytes for load j of an operand (its immediate, j KB, taken back out) and their
  // reduction index in the step; rows and columns beyond the tile's extent are clamped (they only reach outputs that are
  // never stored), reduction indices beyond the range read from outside the buffer: zeros
  unsigned voA[2], voB[2];
  int krA[2], krB[2];
  auto lane_off = [&](bool kc, int j, int ld, int extent, int& kr) -> unsigned {
    unsigned e;
    if (kc) {
      const int r = j * 16 + (lane >> 2);
      kr = ((lane & 3) ^ ((r >> 2) & 3)) * 4;
      e = (unsigned)(min(r, extent - 1) * ld + kr);
    } else {
      const int row = j * 8 + (lane >> 3), c = (lane & 7) * 4;
      kr = row ^ ((row >> 2) & 1);
      e = (unsigned)(kr * ld + (c < extent ? c : 0));
    }
    return e * 4u + 4096u - (unsigned)(j * 1024);
  };
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    voA[j] = lane_off(Op::A_KC, j, (int)o.lda, o.row1 - o.row0, krA[j]);
    voB[j] = lane_off(Op::B_KC, j, (int)o.ldb, N - n0, krB[j]);
  }
  const unsigned lds = (unsigned)(size_t)SYMI_LPTR(ring);
  const float* const b0 = o.B + (Op::B_KC ? n0 * o.ldb : n0);
  auto load = [&](unsigned dst, const float* src, const unsigned (&vo)[2], const int (&kr)[2], int left) {
    const unsigned long long a = (unsigned long long)src - 4096;
    const intx4 rsrc = {__builtin_amdgcn_readfirstlane((int)(unsigned)a), __builtin_amdgcn_readfirstlane((int)((unsigned)(a >> 32) & 0xffffu)),
                        (int)OUTSIDE, 0x00020000};
    const unsigned v0 = kr[0] < left ? vo[0] : OUTSIDE, v1 = kr[1] < left ? vo[1] : OUTSIDE;
    // wait states: of the M0 write, and of a base that came through the vector unit
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %3, 0 offen lds\n\t"
                 "buffer_load_dwordx4 %2, %3, 0 offen offset:1024 lds" ::"s"(dst), "v"(v0), "v"(v1), "s"(rsrc) : "memory");
  };
  auto issue = [&](int t, int st) {
    const int k0 = kbeg + t * F32_CHUNK, left = kend - k0;
    const unsigned dst = lds + st * ((1 + NB) * SO * 4);
    load(dst, o.A + (Op::A_KC ? (long long)k0 : k0 * o.lda), voA, krA, left);
    const float* const sb = b0 + (Op::B_KC ? (long long)k0 : k0 * o.ldb);
#pragma unroll
    for (int j = 0; j < NB; ++j) load(dst + (1 + j) * SO * 4, sb + (j ? (long long)p.f * o.ldb : 0), voB, krB, left);
  };
  floatx16 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  // value 4 s + i is reduction index 8 s + 4 hw + i of the step
  auto read = [&](bool kc, const float* q, float (&x)[8]) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if (kc) {
        const float4 y = *reinterpret_cast<const float4*>(q + r31 * F32_CHUNK + (((2 * s + hw) ^ ((r31 >> 2) & 3)) * 4));
        x[4 * s] = y.x; x[4 * s + 1] = y.y; x[4 * s + 2] = y.z; x[4 * s + 3] = y.w;
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) x[4 * s + i] = q[((8 * s + 4 * hw + i) ^ hw) * 32 + r31];
      }
    }
  };
  const int ns = kbeg < kend ? (kend - kbeg + F32_CHUNK - 1) / F32_CHUNK : 0;
#pragma unroll
  for (int t = 0; t < NST - 1; ++t)
    if (t < ns) issue(t, t);
  int st = 0;
  for (int t = 0; t < ns; ++t) {
    // the loads of step t have landed (with three stages those of the next step may fly), the reads of step t - 1 are through
    if (NST == 3 && t + 1 < ns) __builtin_amdgcn_s_waitcnt(0x0070 + 2 + 2 * NB); else __builtin_amdgcn_s_waitcnt(0x0070);
    asm volatile("" ::: "memory");
    if (t + NST - 1 < ns) issue(t + NST - 1, st == 0 ? NST - 1 : st - 1);
    const float* const q = ring + st * ((1 + NB) * SO);
    float a[8], b[NB][8];
    read(Op::A_KC, q, a);
#pragma unroll
    for (int j = 0; j < NB; ++j) read(Op::B_KC, q + (1 + j) * SO, b[j]);
    floatx16 part[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) part[j][r] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) part[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j][i], part[j], 0, 0, 0);
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][r] += part[j][r];
    asm volatile("" ::: "memory");
    st = st == NST - 1 ? 0 : st + 1;
  }
  auto sum = [&](int w, int j) { return smem + w * RING + j * 32 * LDR; };   // wavefront w's, block j
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) sum(wave, j)[(8 * (r >> 2) + 4 * hw + (r & 3)) * LDR + r31] = acc[j][r];
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 1024 / (64 * NW); ++i) {
    const int e = tid + 64 * NW * i, r = e >> 5, col = n0 + (e & 31);
    if (o.row0 + r >= o.row1 || col >= N) continue;
    float x[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      x[j] = sum(0, j)[r * LDR + (e & 31)];
#pragma unroll
      for (int w = 1; w < NW; ++w) x[j] += sum(w, j)[r * LDR + (e & 31)];
    }
    f32_store<MODE>(p, o.group, o.row0 + r, col, x[0], x[NB - 1]);
  }
}

template <int MODE, int NW>
__global__ __launch_bounds__(64 * NW) void gemm_f32_small_kernel(GemmParams p) {
  __shared__ __attribute__((aligned(1024))) float smem[F32Small<MODE, NW, 1>::LDS];
  f32_small_tile<MODE, NW, 1>(p, blockIdx.x, smem);
}

// Two products that do not need each other, one launch: the weight gradient MODE, whose tiles have the longer reductions, in the first
// `first` workgroups, and an activation gradient (dh beside dW2, dX beside dW1), whose reductions NW wavefronts share.
template <int MODE, int WITH, int NW>
__global__ __launch_bounds__(512) void gemm_f32_small_pair_kernel(GemmParams p, GemmParams q, int first) {
  using A = F32Small<MODE, 8, 1>;
  using B = F32Small<WITH, NW, 8 / NW>;
  static_assert(A::NT == 512 && B::NT == 512 && A::LDS == B::LDS, "one LDS area");
  __shared__ __attribute__((aligned(1024))) float smem[A::LDS];
  if ((int)blockIdx.x < first) f32_small_tile<MODE, 8, 1>(p, blockIdx.x, smem);
  else f32_small_tile<WITH, NW, 8 / NW>(q, blockIdx.x - first, smem);
}

// bf16 forward products, at most 32 rows per slot on average: the tile that streams weights.  Both products against
// the large tile, 32 rows per slot on average, in all slots / half / a quarter / a tenth / one of them (us):
//   96 slots, d = 1024, f = 4096    558 : 624   328 : 359   217 : 228   187 : 171   138 : 124
//   128 slots, d = 2048, f = 1408   505 : 574   308 : 332   209 : 213   176 : 172   121 : 113
//   60 slots, d = 1160, f = 2744    341 : 420   237 : 254   189 : 187   153 : 150   116 : 109
//   40 slots, d = 4096, f = 2048    487 : 605   302 : 340   203 : 195   158 : 162   133 : 157
//   24 slots, d = 256, f = 768       28 : 44     25 : 42     23 : 42     21 : 47     21 : 47
// and 8 on average, in a tenth / one: 112 : 134, 67 : 81; 113 : 124, 46 : 104; 91 : 115, 64 : 109; 91 : 149, 67 : 130;
// 20 : 40, 20 : 48.  The host knows the mean only.  Placement keeps the slots even, where the tile gains 10 - 20 %;
// with every row in a tenth of the slots or fewer, 300 rows and more in each, it loses 2 - 12 % on some
// shapes, so the line lies no higher: 64 rows in every slot of the first shape 349 : 280.
static bool few_rows(const symi_cfg* c) {
  return c->dtype == SYMI_BF16 && (long long)c->T * c->k <= 32LL * c->S_tot;
}

// Whether these tiles come from a table, for both products: the launch that writes it takes 1 - 2 us, finding a tile without it
// about 1 us of every workgroup, which long reductions hide behind each other and short ones do not.  Time counted /
// from the table of the two products together over 250 drawn shapes (8 - 960 slots of 0.1 - 32 rows on average, d 64 - 4096, f
// 128 - 14336), geometric mean by workgroups per compute unit, d <= 256 / <= 640 / above: 0 - 2 0.91, 0.92, 0.94; 2 - 5 0.96, 0.96, 0.96; 5 - 8 1.01, 0.98,
// 0.98; 8 - 14 1.06, 1.01, 1.00; 14 - 20 1.12, 1.04, 1.04; 20 - 40 1.14, 1.07, 1.00; beyond 1.22 (up to 1.53), 1.11, 1.03.
static bool few_rows_table(const symi_ctx* ctx) {
  const symi_cfg* const c = &ctx->cfg;
  return ((long long)c->T * c->k / FEW_BM + c->S_tot) * (cdiv(c->f, 64) + cdiv(c->d, 128)) > 8LL * ctx->cus;
}

// bf16 variable-row products that take the 128 x 128 tile: those of few tiles, where the latency of one tile is the
// time, and those of short reductions with slots of less than a tile, where set-up and epilogue are (two workgroups share a unit
// and hide theirs behind each other).  Long reductions of many tiles belong to the large tile, which loads half as much per
// product and slices a nearly empty last round; so do slots of more rows than one small tile has.  Times large / small over
// 550 drawn shapes (8 - 1024 slots, 20 - 600 rows per slot on average, d 64 - 4096, f 64 - 8192; events around the launch, the
// sum of the slices included), geometric mean (a tenth lies below / above), with replicas as a batch of the same popularity
// before would place them (Zipf or drifted), and misplaced: Zipf 2.4 over even replicas, most rows in a few slots.
//                          first forward      second forward     hidden gradient    input gradient
//   few tiles              1.23 (1.03/1.47)   1.22 (0.95/1.53)   1.31 (0.99/1.74)   1.30 (1.00/1.57)
//     misplaced            1.20 (0.92/1.50)   1.23 (0.94/1.56)   1.35 (1.03/1.81)   1.36 (1.04/1.59)
//   small mean (lines)     1.11 (0.98/1.26)   1.13 (0.97/1.30)   1.14 (1.01/1.31)   1.09 (0.97/1.23)
//     misplaced            0.95 (0.79/1.10)   0.98 (0.81/1.18)   1.09 (0.93/1.29)   0.99 (0.80/1.23)
//   next beyond the lines, where r <= 128, K <= 1024 or r <= 96, K <= 2048 (1792):
//                          0.98 (0.88/1.12)   0.99 (0.89/1.12)   0.99 (0.86/1.10)   0.96 (0.83/1.10)
//     misplaced            0.91 (0.78/1.07)   0.94 (0.81/1.11)   0.97 (0.81/1.12)   0.92 (0.78/1.08)
// At 1 - 1.25 times the limit of tiles x K, 64 - 128 rows: 0.97, 1.01, 1.10, 1.02; at half to all of it, more than 128 rows: 0.94, 0.99,
// 1.06, 1.19, so there it is half as high for the forward products.  The host knows the mean number of rows only.
// All this with one kernel at a time.  Where the weight gradients run beside them on the helper stream, the backward's two
// products leave them less of the chip with this tile, two workgroups to a unit that none of theirs fits beside: expert backward
// large / small over 150 drawn shapes, by T*k*d*f: below 3.5e8 1.07, to 7e8 1.05, to 3e9 1.03 (0.93 - 1.13), beyond 1.00 (0.88 - 1.08;
// 256 rows and more on average 0.94: E = 16, k = 6, d = 240, f = 536, 52578 rows 340 : 375 us).  So not from 3e9 on, and the input
// gradient not in more than two rounds of tiles (six shapes with 2.2 - 5.6 rounds 0.92 - 0.97, one to two rounds 1.00 - 1.16).
// No reduction that the large tile may slice (from 32 steps on), so that no result depends on the tile.
static bool mid_tile(const symi_ctx* ctx, int mode) {
  const symi_cfg* const c = &ctx->cfg;
  if (c->dtype != SYMI_BF16 || mode > BWD_DX || ((mode == FWD1 || mode == FWD2) && few_rows(c))) return false;
  const long long A = (long long)c->T * c->k, S = c->S_tot;
  if (A / MID_BM + S > 65535) return false;   // its row tiles are a grid.y coordinate
  const int K = mode == FWD1 || mode == BWD_DH ? c->d : mode == FWD2 ? c->f : 2 * c->f;
  const int ntx = mode == FWD1 ? cdiv(c->f, 64) : cdiv(mode == BWD_DH ? c->f : c->d, 128);
  const long long tiles = std::max(A / MID_BM + S / 2, S) * ntx;
  if (mode >= BWD_DH && ctx->side && ((double)A * c->d * c->f >= 3e9 || (mode == BWD_DX && tiles > 4LL * ctx->cus))) return false;
  // mean rows and reduction length, up to three lines for each product
  constexpr int LINES[4][3][2] = {{{64, 1536}, {112, 640}}, {{64, 1984}, {112, 1024}}, {{40, 1792}, {80, 1536}, {128, 512}}, {{48, 1536}, {96, 640}}};
  for (const auto& line : LINES[mode])
    if (A <= line[0] * S && K <= line[1]) return true;
  const long long work = tiles * K * (mode <= FWD2 && A > 128 * S ? 2 : 1);
  return mode == FWD1 || mode == BWD_DH ? work <= 1 << 19 : work <= 3 << 17 && K <= 1984;
}

// Whether the 128 x 128 tiles of a product come from a table: as with the small-batch tile, counting takes about a microsecond of
// every workgroup.  Counted / table, us: 224 slots of 90 rows, d = 160, f = 11768 (68448 workgroups) first forward product 1032 : 912, hidden
// gradient 691 : 649; 128 of 100, d = 312, f = 7048 (25308) 505 : 465, 340 : 328; 160 of 100, d = 512, f = 2048 (9120) 210 : 206,
// 156 : 155; below 16 per unit a launch that would write it takes longer than it saves.
static bool mid_table(const symi_ctx* ctx, int mode) {
  const symi_cfg* const c = &ctx->cfg;
  if (!mid_tile(ctx, mode)) return false;
  const int ntx = mode == FWD1 ? cdiv(c->f, 64) : cdiv(mode == BWD_DH ? c->f : c->d, 128);
  return ((long long)c->T * c->k / MID_BM + c->S_tot) * ntx > 16LL * ctx->cus;
}

// Short weight gradients (gemm_duo_kernel), by the mean: up to 96 rows per class (or slot) 1.05 (0.94 - 1.17) over 50 drawn backwards, 100 - 144 rows
// 1.01 (0.97 - 1.06), beyond 0.98 and below.  On the helper stream beside a large tile, which needs a whole unit and waits until both of its
// workgroups are through, up to 1 GiB of gradients: below that 42 drawn layers 1.03 (0.97 - 1.14), beyond it the waiting costs more than the tile
// saves (64 classes of d = 1848, f = 1456, 1516 rows, step 1996 : 2066 us, 128 of 232, 11624, 4824 rows 4120 : 4229).
static bool short_gradients(const symi_ctx* ctx, bool per_slot) {
  const symi_cfg* const c = &ctx->cfg;
  if (ctx->side && !mid_tile(ctx, BWD_DX) && 12LL * (per_slot ? c->S_tot : c->E) * c->d * c->f > 1LL << 30) return false;
  return c->dtype == SYMI_BF16 && (long long)c->T * c->k <= 96LL * (per_slot ? c->S_tot : c->E) && cdiv(std::max(2 * c->f, c->d), DUO_BM) <= 65535;
}

// fp32: the shared reduction, by the count of 64 x 128 tiles (variable rows: about half a tile of padding per slot).  Below one round of them the shared
// reduction, whose time is the latency of a tile; beyond it the split one.  A class's weight gradient reduces over up to T
// rows, and the most popular class makes the longest chain there is, which the shared reduction cuts in eight: there up to
// two rounds (24 classes, d = 80, f = 376, 4940 tokens: step 232 -> 167 us, 24 classes of d = 280, f = 512 backward 184 ->
// 142), but not for single slots, which placement keeps even (36 slots of 352 rows, d = 184, f = 288 169 : 177).  Groups of
// a few rows are bound by their stores, which the fp32 tile has more of in flight: slots of 1 - 5 rows 164 : 172 (54 slots
// of d = 312, f = 992), 86 : 90 (32 slots of d = 296, f = 552), the split one from some 16 rows on.
static bool f32_small(const symi_ctx* ctx, int mode, bool per_slot) {
  const symi_cfg* const c = &ctx->cfg;
  const bool varm = mode <= BWD_DX;
  const int cols = mode == FWD1 || mode == BWD_DH || mode == WGRAD2 ? c->f : c->d;
  const long long A = (long long)c->T * c->k, groups = per_slot ? c->S_tot : c->E;
  const long long rows = varm ? A / F32_BM + c->S_tot / 2 : cdiv(mode == WGRAD1 ? 2 * c->f : c->d, F32_BM) * groups;
  return rows * cdiv(cols, mode == FWD1 ? 64 : 128) < (!varm && !per_slot && A >= 64 * groups ? 2 : 1) * ctx->cus;
}

template <int MODE>
static unsigned f32_small_tiles(const symi_cfg* c, const GemmParams& p) {
  const long long ntx = cdiv(MODE == FWD1 ? c->f : p.N, 32);
  return (unsigned)(ntx * (MODE <= BWD_DX ? (long long)c->T * c->k / 32 + c->S_tot : (long long)cdiv(p.M, 32) * (p.per_slot ? c->S_tot : c->E)));
}

// Eight wavefronts share a reduction of dh or dX where its tiles then all run at once, two workgroups to a unit: 8 classes of
// d = 64, f = 864, 848 rows, backward 46 us with eight, 55 with four; d = 232, f = 336, 156 rows, step 63 : 74; beyond, four (two tiles to a
// workgroup beside a weight gradient): c1's dh and dW2 17.0 with eight, 12.4.  The same rule one by one and in pairs, and so the same bits.
static bool f32_share_eight(const symi_ctx* ctx, int n_cols) {
  return cdiv(n_cols, 32) * ((long long)ctx->cfg.T * ctx->cfg.k / 32 + ctx->cfg.S_tot / 2) < 2LL * ctx->cus;
}

// fp32: do any of these products read the table of row tiles or the order of the classes?
static bool f32_table(const symi_ctx* ctx, std::initializer_list<int> modes, bool per_slot) {
  for (int m : modes)
    if (!f32_small(ctx, m, per_slot)) return true;
  return false;
}

template <int MODE>
static void launch_gemm(const symi_ctx* ctx, const GemmParams& p, int n_cols, int max_mtiles,
                        hipStream_t st) {
  const symi_cfg* const cfg = &ctx->cfg;
  if (cfg->dtype == SYMI_BF16) {
    if constexpr (MODE == FWD1 || MODE == FWD2) {
      if (few_rows(cfg)) {
        dim3 grid(cdiv(n_cols, MODE == FWD1 ? 64 : 128), cfg->T * cfg->k / FEW_BM + cfg->S_tot);
        if (few_rows_table(ctx))
          SYMI_TIMED(ctx, K_GEMM_FWD1 + MODE, st, (gemm_few_rows_kernel<MODE, true><<<grid, GT, 0, st>>>(p)));
        else
          SYMI_TIMED(ctx, K_GEMM_FWD1 + MODE, st, (gemm_few_rows_kernel<MODE, false><<<grid, GT, 0, st>>>(p)));
        return;
      }
    }
    if constexpr (MODE <= BWD_DX) {
      if (mid_tile(ctx, MODE)) {
        dim3 grid(cdiv(n_cols, MODE == FWD1 ? 64 : 128), cfg->T * cfg->k / MID_BM + cfg->S_tot);
        if (mid_table(ctx, MODE))
          SYMI_TIMED(ctx, K_GEMM_FWD1 + MODE, st, (gemm_mid_kernel<MODE, true><<<grid, GT, 0, st>>>(p)));
        else
          SYMI_TIMED(ctx, K_GEMM_FWD1 + MODE, st, (gemm_mid_kernel<MODE, false><<<grid, GT, 0, st>>>(p)));
        return;
      }
    }
    const int bn = MODE == FWD1 ? BN / 2 : BN;
    const int ntx = cdiv(n_cols, bn);
    if constexpr (MODE >= WGRAD2) {
      if (short_gradients(ctx, p.per_slot)) {
        const int groups = p.per_slot ? cfg->S_tot : cfg->E;
        SYMI_TIMED(ctx, K_GEMM_FWD1 + MODE, st, (gemm_duo_kernel<MODE><<<dim3(ntx, cdiv(p.M, DUO_BM), groups), GT, 0, st>>>(p)));
        return;
      }
    }
    // FWD2, BWD_DX: room for the slices of the last round's tiles (at most cus workgroups more)
    const bool may_slice = (MODE == FWD2 || MODE == BWD_DX) && p.partials && cdiv(p.K, BK) / 16 >= 2;
    const int extra = may_slice ? cdiv(p.cus, ntx) : 0;
    dim3 grid(ntx, MODE <= BWD_DX ? max_mtiles + extra : cdiv(p.M, BM), MODE <= BWD_DX ? 1 : (p.per_slot ? cfg->S_tot : cfg->E));
    SYMI_TIMED(ctx, K_GEMM_FWD1 + MODE, st, (gemm_bf16_kernel<MODE><<<grid, GT, 0, st>>>(p)));
    if (may_slice)   // the sliced round holds at most cus / 2 tiles
      SYMI_TIMED(ctx, K_SLICE_SUM, st, (slice_sum_kernel<<<dim3(BM / 16, std::max(1, p.cus / 2)), 256, 0, st>>>(p, ntx)));
  } else {
    constexpr bool VARM = MODE <= BWD_DX;
    const int groups = p.per_slot ? cfg->S_tot : cfg->E;
    if (f32_small(ctx, MODE, p.per_slot)) {
      const unsigned n = f32_small_tiles<MODE>(cfg, p);
      if constexpr (MODE >= BWD_DH) {
        if (MODE > BWD_DX || f32_share_eight(ctx, n_cols)) {
          SYMI_TIMED(ctx, K_GEMM_FWD1 + MODE, st, (gemm_f32_small_kernel<MODE, 8><<<n, 512, 0, st>>>(p)));
          return;
        }
      }
      if constexpr (MODE <= BWD_DX) SYMI_TIMED(ctx, K_GEMM_FWD1 + MODE, st, (gemm_f32_small_kernel<MODE, 4><<<n, 256, 0, st>>>(p)));
      return;
    }
    const int ntx = cdiv(n_cols, 128);
    if constexpr (!VARM) {
      if ((long long)cfg->T * cfg->k < 16LL * groups) {
        SYMI_TIMED(ctx, K_GEMM_FWD1 + MODE, st, (gemm_f32_kernel<MODE><<<dim3(ntx, cdiv(p.M, F32_BM), groups), 256, 0, st>>>(p)));
        return;
      }
    }
    const long long cols = cdiv(n_cols, MODE == FWD1 ? F32S_T / 2 : F32S_T);
    const long long tiles = cols * (VARM ? (long long)cfg->T * cfg->k / F32S_T + cfg->S_tot : (long long)cdiv(p.M, F32S_T) * groups);
    SYMI_TIMED(ctx, K_GEMM_FWD1 + MODE, st,
               (gemm_f32_split_kernel<MODE><<<(unsigned)std::min(tiles, 3LL * ctx->cus), 256, 0, st>>>(p, groups)));
  }
}

template <int MODE, int WITH>
static void launch_f32_pair(const symi_ctx* ctx, const GemmParams& p, const GemmParams& q, hipStream_t st) {
  const symi_cfg* const c = &ctx->cfg;
  const unsigned first = f32_small_tiles<MODE>(c, p), n = f32_small_tiles<WITH>(c, q);
  if (f32_share_eight(ctx, q.N))
    gemm_f32_small_pair_kernel<MODE, WITH, 8><<<first + n, 512, 0, st>>>(p, q, (int)first);
  else
    gemm_f32_small_pair_kernel<MODE, WITH, 4><<<first + (n + 1) / 2, 512, 0, st>>>(p, q, (int)first);
}

// logits = X Wr^T + b, bf16 (symi_router_fwd).  Streams X once in 64-token tiles, two stages ahead; bound by the latency of
// d / 64 steps where the tiles do not fill the chip, by memory beyond.  Against 128-token tiles through registers with two
// barriers per step, us: T = 5573, E = 128, d = 2896 48 -> 28; 464, 16, 720 16 -> 10; 16384, 8, 4096 57 -> 34; 32768, 64, 2048
// 41 -> 29; 65536, 128, 4096 157 -> 155.  Same bits.
void launch_router_fwd(const symi_ctx* ctx, const void* X, const void* Wr, const float* b, float* logits, hipStream_t st) {
  GemmParams p = {};
  p.A = X; p.B = Wr; p.C = logits; p.UV = b;
  p.M = ctx->cfg.T; p.N = ctx->cfg.E; p.K = ctx->cfg.d;
  SYMI_TIMED(ctx, K_ROUTER_FWD, st, (gemm_few_rows_kernel<GATE, false><<<dim3(cdiv(p.M, FEW_BM), cdiv(p.N, 128)), GT, 0, st>>>(p)));
}

// where sliced reductions keep their partial tiles (bf16 configurations only)
static void set_split(const symi_ctx* ctx, void* ws, GemmParams& p) {
  p.cus = std::min(ctx->cus, SPLIT_CUS);
  p.partials = ctx->slicing && ctx->cfg.dtype == SYMI_BF16
                   ? reinterpret_cast<float*>(static_cast<char*>(ws) + ctx->L.split_part) : nullptr;
}

}  // namespace symi

using namespace symi;

extern "C" int symi_expert_fwd(const symi_ctx* ctx, const void* Xp, const int32_t* slot_offsets,
                               const void* W1_slots, const void* W2_slots, void* UV, void* H,
                               void* Yp, void* ws, void* stream) {
  SYMI_ENTER(ctx, "symi_expert_fwd");
  const long long A = (long long)cfg->T * cfg->k;
  if (A == 0) return SYMI_OK;
  SYMI_REQUIRE(Xp && slot_offsets && W1_slots && W2_slots && UV && H && Yp && ws, "symi_expert_fwd",
               "NULL pointer");
  hipStream_t st = as_stream(stream);
  const WsLayout& L = ctx->L;
  int32_t* map = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + L.tile_map);
  int32_t* map128 = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + L.tile_map128);
  const int max_mtiles = (int)(A / GEMM_BM) + cfg->S_tot;
  TileMaps maps = {};
  if (cfg->dtype == SYMI_F32 ? f32_table(ctx, {FWD1, FWD2}, false) : few_rows(cfg) && few_rows_table(ctx)) maps.of64 = map;
  if (cfg->dtype == SYMI_BF16 && !few_rows(cfg)) {
    if (!(mid_tile(ctx, FWD1) && mid_tile(ctx, FWD2))) maps.of256 = map;
    if (mid_table(ctx, FWD1) || mid_table(ctx, FWD2)) maps.of128 = map128;
  }
  if (maps.of256 || maps.of128 || maps.of64)
    SYMI_TIMED(ctx, K_TILE_MAP, st, (tile_map_kernel<<<1, 256, 0, st>>>(slot_offsets, nullptr, cfg->S_tot, cfg->E, maps, nullptr)));

  GemmParams p = {};
  p.tile_map = map;
  p.tile_map128 = map128;
  p.slot_offsets = slot_offsets;
  p.n_slots = cfg->S_tot;
  set_split(ctx, ws, p);
  p.d = cfg->d;
  p.f = cfg->f;
  // u|v = Xp W1^T, h = silu(u)*v
  p.A = Xp; p.B = W1_slots; p.UVout = UV; p.H = H;
  p.b_group_stride = 2LL * cfg->f * cfg->d;
  p.N = cfg->f; p.K = cfg->d;
  launch_gemm<FWD1>(ctx, p, cfg->f, max_mtiles, st);
  // Yp = h W2^T
  p.A = H; p.B = W2_slots; p.C = Yp;
  p.b_group_stride = (long long)cfg->d * cfg->f;
  p.N = cfg->d; p.K = cfg->f;
  launch_gemm<FWD2>(ctx, p, cfg->d, max_mtiles, st);
  SYMI_LAUNCH_CHECK("symi_expert_fwd");
  return SYMI_OK;
}

// The backward's five products form two chains that only meet at du|dv:
//   dh -> du|dv -> dXp          and          dW2 (needs dYp, H only) -> dW1 (needs du|dv)
// Run back to back each launch rounds its tile count up to whole rounds of 256 workgroups
// (config c2: 296 tiles of the dXp product are two rounds, the second one 84 % empty) and
// the store-bound zero tiles of the weight gradients never meet the MFMA-bound tiles.  The
// second chain is therefore enqueued on the context's helper stream (created by symi_create
// when the flags allow it, the products or their gradients are large enough and the dXp product has
// fewer than 8 rounds of tiles; default priority, non-blocking), forked from and joined back into the caller's stream with events,
// so workgroups of both chains share the chip.  Otherwise everything stays on the caller's
// stream, in order.

// per_slot = false: dW1_out / dW2_out are per class (all replica slots summed in the GEMM);
// per_slot = true: one gradient per replica slot (its own rows only)
static int expert_bwd_impl(const char* who, const symi_ctx* ctx, const void* dYp, const void* Xp,
                           const void* UV, const void* H, const int32_t* slot_offsets,
                           const int32_t* first_slot, const void* W1_slots, const void* W2_slots,
                           void* dXp, float* dW1_class, float* dW2_class, void* ws, void* stream,
                           bool per_slot, bool skip_empty = false) {
  SYMI_ENTER(ctx, who);
  const long long A = (long long)cfg->T * cfg->k;
  SYMI_REQUIRE(slot_offsets && first_slot && dW1_class && dW2_class && ws, who, "NULL pointer");
  SYMI_REQUIRE(A == 0 || (dYp && Xp && UV && H && W1_slots && W2_slots && dXp), who, "NULL pointer");
  hipStream_t st = as_stream(stream);
  const WsLayout& L = ctx->L;
  int32_t* map = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + L.tile_map);
  int32_t* map128 = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + L.tile_map128);
  void* dUV = static_cast<char*>(ws) + L.duv;
  const int max_mtiles = (int)(A / GEMM_BM) + cfg->S_tot;

  int32_t* order = reinterpret_cast<int32_t*>(static_cast<char*>(ws) + L.class_order);
  GemmParams p = {};
  p.tile_map = map;
  p.tile_map128 = map128;
  p.slot_offsets = slot_offsets;
  p.n_slots = cfg->S_tot;
  p.first_slot = first_slot;
  p.class_order = order;
  p.per_slot = per_slot ? 1 : 0;
  p.skip_empty = skip_empty ? 1 : 0;
  set_split(ctx, ws, p);
  p.d = cfg->d;
  p.f = cfg->f;
  TileMaps maps = {};
  // The order of the classes matters to the gradients' last round only; short ones of a small batch go without it, and
  // without a launch where no product reads a table (some 4 us: slot gradients of E = 16, d = 168, f = 584, 98 rows 44 -> 41 us).  Ordered : not, backward
  // of drawn layers whose launch it is, by rows: up to 2560 1.05 (0.99 - 1.07), to 4096 1.02, the gain of 3 - 4 % where the classes are even, 0.89 - 0.98 in
  // four of 40, with a few popular ones (64 classes of d = 368, f = 552, 4052 rows, the most popular with a quarter of them, 104 : 118 us), to 9200
  // 1.01 (0.88 - 1.10): the launch is a smaller part, the late long reduction a larger one.
  bool ordered = !per_slot;
  if (cfg->dtype == SYMI_F32) {
    if (f32_table(ctx, {BWD_DH, BWD_DX, WGRAD2, WGRAD1}, per_slot)) maps.of64 = map;
    else ordered = false;
  } else {
    if (!(mid_tile(ctx, BWD_DH) && mid_tile(ctx, BWD_DX))) maps.of256 = map;
    if (mid_table(ctx, BWD_DH) || mid_table(ctx, BWD_DX)) maps.of128 = map128;
    if (short_gradients(ctx, per_slot) && A <= 4096 && !maps.of256 && !maps.of128) ordered = false;
  }
  if (!ordered) p.class_order = nullptr;
  if (ordered || maps.of256 || maps.of128 || maps.of64)
    SYMI_TIMED(ctx, K_TILE_MAP, st, (tile_map_kernel<<<1, 256, 0, st>>>(slot_offsets, ordered ? first_slot : nullptr, cfg->S_tot, cfg->E, maps, order)));
  // worth it only while a product is a few rounds of workgroups: with many rounds the chip is
  // full anyway and two kernels sharing it only disturb each other's L2 locality; and not for the
  // smallest, where fork, hand-over and join take longer than what they hide (symi_create
  // decides; the context then holds the helper stream)
  const bool side = ctx->side != nullptr && A > 0;
  hipStream_t sw = st;   // stream of the weight-gradient chain
  if (side) {
    if (hipEventRecord(ctx->fork, st) != hipSuccess || hipStreamWaitEvent(ctx->side, ctx->fork, 0) != hipSuccess) {
      set_error("%s: forking onto the helper stream failed", who);
      return SYMI_EHIP;
    }
    sw = ctx->side;
  }
  // class gradients (classes without rows get zeros: their reduction is empty)
  GemmParams pw = p, pw1 = p;
  pw.A = dYp; pw.B = H; pw.C = dW2_class;
  pw.c_group_stride = (long long)cfg->d * cfg->f;
  pw.M = cfg->d; pw.N = cfg->f;
  pw1.A = dUV; pw1.B = Xp; pw1.C = dW1_class;
  pw1.c_group_stride = 2LL * cfg->f * cfg->d;
  pw1.M = 2 * cfg->f; pw1.N = cfg->d;
  // dh = dYp W2, turned into du, dv in the epilogue (dh itself never reaches memory)
  GemmParams px = p;
  p.A = dYp; p.B = W2_slots; p.C = dUV; p.UV = UV;
  p.b_group_stride = (long long)cfg->d * cfg->f;
  p.N = cfg->f; p.K = cfg->d;
  // dXp = dUV W1
  px.A = dUV; px.B = W1_slots; px.C = dXp;
  px.b_group_stride = 2LL * cfg->f * cfg->d;
  px.N = cfg->d; px.K = 2 * cfg->f;
  // small fp32 products of both chains go in pairs (one by one where every launch is timed)
  const bool pairs = cfg->dtype == SYMI_F32 && A > 0 && !side && !ctx->timing;
  const bool pair2 = pairs && f32_small(ctx, BWD_DH, per_slot) && f32_small(ctx, WGRAD2, per_slot);
  const bool pair1 = pairs && f32_small(ctx, BWD_DX, per_slot) && f32_small(ctx, WGRAD1, per_slot);
  if (pair2)
    launch_f32_pair<WGRAD2, BWD_DH>(ctx, pw, p, st);
  else
    launch_gemm<WGRAD2>(ctx, pw, cfg->f, 0, sw);
  if (A > 0) {
    if (!pair2) launch_gemm<BWD_DH>(ctx, p, cfg->f, max_mtiles, st);
    if (side) {   // du|dv is complete: the other chain may go on to dW1
      if (hipEventRecord(ctx->mid, st) != hipSuccess || hipStreamWaitEvent(ctx->side, ctx->mid, 0) != hipSuccess) {
        set_error("%s: event hand-over between the two streams failed", who);
        return SYMI_EHIP;
      }
    }
    if (!pair1) launch_gemm<BWD_DX>(ctx, px, cfg->d, max_mtiles, st);
  }
  if (pair1)
    launch_f32_pair<WGRAD1, BWD_DX>(ctx, pw1, px, st);
  else
    launch_gemm<WGRAD1>(ctx, pw1, cfg->d, 0, sw);
  if (side) {
    if (hipEventRecord(ctx->join, ctx->side) != hipSuccess || hipStreamWaitEvent(st, ctx->join, 0) != hipSuccess) {
      set_error("%s: joining the helper stream failed", who);
      return SYMI_EHIP;
    }
  }
  SYMI_LAUNCH_CHECK(who);
  return SYMI_OK;
}

extern "C" int symi_expert_bwd(const symi_ctx* ctx, const void* dYp, const void* Xp, const void* UV,
                               const void* H, const int32_t* slot_offsets, const int32_t* first_slot,
                               const void* W1_slots, const void* W2_slots, void* dXp,
                               float* dW1_class, float* dW2_class, void* ws, void* stream) {
  return expert_bwd_impl("symi_expert_bwd", ctx, dYp, Xp, UV, H, slot_offsets, first_slot, W1_slots,
                         W2_slots, dXp, dW1_class, dW2_class, ws, stream, false);
}

extern "C" int symi_expert_bwd_active(const symi_ctx* ctx, const void* dYp, const void* Xp,
                                      const void* UV, const void* H, const int32_t* slot_offsets,
                                      const int32_t* first_slot, const void* W1_slots,
                                      const void* W2_slots, void* dXp, float* dW1_class,
                                      float* dW2_class, void* ws, void* stream) {
  return expert_bwd_impl("symi_expert_bwd_active", ctx, dYp, Xp, UV, H, slot_offsets, first_slot,
                         W1_slots, W2_slots, dXp, dW1_class, dW2_class, ws, stream, false, true);
}

extern "C" int symi_expert_bwd_slots(const symi_ctx* ctx, const void* dYp, const void* Xp,
                                     const void* UV, const void* H, const int32_t* slot_offsets,
                                     const int32_t* first_slot, const void* W1_slots,
                                     const void* W2_slots, void* dXp, float* dW1_slot,
                                     float* dW2_slot, void* ws, void* stream) {
  return expert_bwd_impl("symi_expert_bwd_slots", ctx, dYp, Xp, UV, H, slot_offsets, first_slot,
                         W1_slots, W2_slots, dXp, dW1_slot, dW2_slot, ws, stream, true);
}

// ---------------------------------------------------------------- replica all-reduce
// The intra-rank part of the paper's all-reduce (Sec. 4.1): for every class the first of its
// slots is the representative; the other slots add their gradient to it (slot order), the
// sum is scaled and copied back to all of them.  16 bytes per lane, one class per blockIdx.y.  ONCE: every gradient is read
// once, past the caches' replacement order, where together they outgrow the 256 MB memory-side cache.  Behind the products that
// wrote them, time plain / so over 160 drawn shapes by the size of all slots' gradients: up to 256 MB 1.00 (0.92 - 1.06), 256 - 512 MB
// 1.02, 512 - 1024 1.08, beyond 1.12 (1.02 - 1.25); us: 728 : 635 (32 slots of d = 1128, f = 6376), 202 : 162 (64 of d = f = 1024), 725 : 705 (96 of
// 1024, 4096), 1621 : 1636 (128 of 2048, 1408, every class twice).
namespace symi {
template <bool ONCE>
__global__ __launch_bounds__(256) void replica_allreduce_kernel(float4* __restrict__ g,
                                                                const int32_t* __restrict__ first_slot,
                                                                long long n4, float scale) {
  const int e = blockIdx.y;
  const int q0 = first_slot[e], q1 = first_slot[e + 1];
  if (q1 - q0 == 1 && scale == 1.f) return;   // a single replica: nothing to exchange
  for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n4; i += (long long)gridDim.x * 256) {
    auto load = [&](int q) {
      const floatx4* const at = reinterpret_cast<const floatx4*>(g) + (long long)q * n4 + i;
      return ONCE ? __builtin_nontemporal_load(at) : *at;
    };
    floatx4 a = load(q0);
    for (int q = q0 + 1; q < q1; ++q) a += load(q);
    a *= scale;
    for (int q = q0; q < q1; ++q) reinterpret_cast<floatx4*>(g)[(long long)q * n4 + i] = a;
  }
}
}  // namespace symi

extern "C" int symi_replica_allreduce(const symi_ctx* ctx, const int32_t* first_slot, float scale,
                                      float* dW1_slot, float* dW2_slot, void* stream) {
  SYMI_ENTER(ctx, "symi_replica_allreduce");
  SYMI_REQUIRE(first_slot && dW1_slot && dW2_slot, "symi_replica_allreduce", "NULL pointer");
  hipStream_t st = as_stream(stream);
  const long long n1 = 2LL * cfg->f * cfg->d / 4, n2 = (long long)cfg->d * cfg->f / 4;
  auto blocks = [](long long n4) { long long b = (n4 + 255) / 256; return (unsigned)(b > 2048 ? 2048 : (b < 1 ? 1 : b)); };
  const auto kernel = 16LL * (n1 + n2) * cfg->S_tot > 256LL << 20 ? replica_allreduce_kernel<true> : replica_allreduce_kernel<false>;
  SYMI_TIMED(ctx, K_REPLICA_AR, st, (kernel<<<dim3(blocks(n1), cfg->E), 256, 0, st>>>(
      reinterpret_cast<float4*>(dW1_slot), first_slot, n1, scale)));
  SYMI_TIMED(ctx, K_REPLICA_AR, st, (kernel<<<dim3(blocks(n2), cfg->E), 256, 0, st>>>(
      reinterpret_cast<float4*>(dW2_slot), first_slot, n2, scale)));
  SYMI_LAUNCH_CHECK("symi_replica_allreduce");
  return SYMI_OK;
}
