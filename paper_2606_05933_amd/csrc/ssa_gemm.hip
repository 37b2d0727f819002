// HIP kernels for gfx950 of the dense steps of a transformer layer
// (include/ssa_layer.h): the linear layers as one MFMA GEMM with fused
// epilogues, and RMSNorm.
//
// ssa_linear: out = x W^T, x [M, K] and W [N, K] bf16, both K-contiguous (the
// torch Linear layout), fp32 accumulation.
//  * One workgroup per output tile and K range.  A tile configuration
//    (TileCfg) sets the wave grid and each wave's share in
//    v_mfma_f32_16x16x32_bf16 tiles; the host picks one per shape.
//  * W is the MFMA A operand (MFMA rows = output columns n) and x the B operand
//    (MFMA columns = tokens), so a lane ends with 4 consecutive n of one token:
//    one 8-byte store per 16 x 16 tile.
//  * K blocks of 64 are copied global -> LDS without registers
//    (global_load_lds_dwordx4, a scalar row base and one 32-bit lane offset)
//    into a ring of STAGES stages; one barrier per block.  LDS rows are 128
//    bytes; the 16-byte chunk c of row r sits at chunk c ^ (r & 7), so the 16
//    rows one ds_read_b128 reads fall on 8 distinct chunk slots per lane octet
//    (no bank conflict).
//  * The loop is software-pipelined over the two K halves of a block: while the
//    MFMAs of one half run, the fragments of the next half are read, across the
//    barrier too (it sits between a block's halves, where the next block has
//    landed and this block's reads are done, so its stage is refilled at once),
//    and the copies go out one by one between the rows of MFMAs.  Reading a
//    block's fragments only after its barrier left the matrix cores idle for
//    the LDS reads of every block (4096 x 4096 x 14336 with the residual: 397 us,
//    360 with this loop and the tiles chosen by plan_cost).
//  * Rows of x past M are read from the 8-row piece of row M - 1 (in bounds) and
//    never stored.
//  * With one M tile, W is read once by the whole chip: its copies carry the
//    non-temporal hint, and tile t starts its K loop at block 3 t so that
//    neighbouring tiles, whose rows are a power of two apart, do not all walk the
//    same memory channels.  24 x 28672 x 4096 with W out of the caches, as a
//    model's weights are: 37.1 us (6.3 TB/s); without the stagger 39.2, without the
//    hint 42.2, with neither 44.6.  A call repeated on weights that the last-level
//    cache could hold loses by the hint (128 x 28672 x 4096: 47.5 us, 37.5
//    without); a decoder layer of 128 decodes takes 272 us with it and 280 without
//    it past 32 rows.  With several M tiles neither: they share W and x panels
//    through the caches, which wants them on the same K block.
//  * Too few tiles to fill the chip: K is split; each split writes its fp32
//    tile with device-scope stores, takes a ticket, and the last one adds the
//    splits in split order (the result does not depend on arrival order),
//    applies the epilogue and resets the ticket.  Merging neighbours pairwise up
//    a tree instead (each workgroup reads at most log2(splits) tiles) measured
//    slower: a level costs a store, a ticket and a read one after the other
//    (24 x 4096 x 14336 in 4 splits: 35 against 23.5 us).
//  * Work ids are laid out so that consecutive ids run on one XCD and share its
//    L2: groups of M tiles by N tiles.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "../../include/ssa_layer.h"
#include "ssa_device.h"
#include "ssa_layer_internal.h"

namespace {
using namespace ssa_dev;

constexpr int kNormThreads = 256;
constexpr int BK = 64;  // K block: one 128-byte LDS row per operand row
constexpr int kXcds = 8;
constexpr float kLog2e = 1.4426950408889634f;
// Rows this long take 64-bit lane addresses: 7 rows of 2 K bytes and a chunk pass
// 32 bits not far above.
constexpr int kWideK = 1 << 28;
// Split tickets at the start of the workspace.
constexpr size_t kTicketBytes = ssa::kLinearTicketBytes;
constexpr int kTicketWords = (int)kTicketBytes / 4;

// Reads of the partials: 16-byte buffer loads with the device-coherent cache
// policy (sc1), the instruction of a device-scope load, so they do not hit a
// stale line of this XCD's L2.  Being plain loads to the compiler, they are
// issued back to back and waited for where a value is used (device-scope
// atomic loads would be serialised).  Offsets are bytes from the tile's first
// partial; a read past num_records would return zeros, never fault.
struct PartReader {
  __amdgpu_buffer_rsrc_t rsrc;
  __device__ explicit PartReader(const float* base)
      : rsrc(__builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(base), (short)0, 0x7fffffff,
                                               0x00020000)) {}
  __device__ f32x4 operator()(int byte_off) const {
    return __builtin_bit_cast(
        f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, byte_off, 0, kCachePolicySc1));
  }
};

// silu(z) = z / (1 + e^-z), with e^-z as 2^(-z log2 e)
__device__ __forceinline__ float silu(float z) {
  return z * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-z * kLog2e));
}

struct GemmArgs {
  const uint16_t* x;
  const uint16_t* w;
  const uint16_t* res;
  uint16_t* out;
  uint32_t* tickets;
  float* part;
  int m, n, k;
  int tiles_m, tiles_n, splits, kbps, kblocks, group;
};

// A tile configuration: NWM x NWN waves, each owning TM x TN MFMA tiles of
// 16 x 16 (TM along tokens, TN along output features); STAGES K blocks in the
// LDS ring; OCC workgroups per CU the launch bounds ask for.
template <int NWM_, int NWN_, int TM_, int TN_, int STAGES_, int OCC_>
struct TileCfg {
  static constexpr int NWM = NWM_, NWN = NWN_, TM = TM_, TN = TN_, STAGES = STAGES_, OCC = OCC_;
  static constexpr int kWaves = NWM * NWN, kThreads = kWaves * 64;
  static constexpr int BM = NWM * TM * 16, BN = NWN * TN * 16;
  static constexpr int kStage = (BM + BN) * BK * 2;  // x rows, then W rows
  static constexpr int kPieces = (BM + BN) / 8;      // 1 KB copies (8 rows) per stage
  static constexpr int kLoads = kPieces / kWaves;    // copies per wave per stage
  static constexpr int kTileFloats = BM * BN;
  static constexpr bool kRoll = TM >= 4;             // x fragments replaced row by row
  static_assert(kPieces % kWaves == 0, "copies must split evenly over the waves");
  static_assert(TN % 2 == 0, "the SwiGLU epilogue pairs n tiles");
  static_assert(OCC * STAGES * kStage <= 160 * 1024, "LDS of a CU");
  static_assert((STAGES - 1) * kLoads < 64, "vmcnt range");
};

// Wait until at most min(left, MAX) K blocks (LOADS copies each) of this wave
// are in flight.
template <int MAX, int LOADS>
__device__ __forceinline__ void wait_blocks(int left) {
  if constexpr (MAX <= 0) {
    vm_wait<0>();
  } else {
    if (left >= MAX) vm_wait<MAX * LOADS>();
    else wait_blocks<MAX - 1, LOADS>(left);
  }
}

// Barrier of a K block: this wave's LDS reads have returned, and no memory
// access moves across (copies in flight stay in flight).
__device__ __forceinline__ void block_barrier() {
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// MODE: kShared, several M tiles; kStream, one M tile (W copies with the
// non-temporal hint, staggered K loops); kWide, rows too long for a 32-bit lane
// offset (7 rows of 2 K bytes): 64-bit lane addresses.
enum { kShared, kStream, kWide };
template <class C, int EPI, int MODE>
__global__ __launch_bounds__(C::kThreads, C::OCC) void linear_kernel(GemmArgs a) {
  constexpr int TM = C::TM, TN = C::TN, STAGES = C::STAGES, LOADS = C::kLoads;
  constexpr int BM = C::BM, BN = C::BN;
  __shared__ __attribute__((aligned(16))) char lds[STAGES * C::kStage];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w / C::NWN, wn = w % C::NWN;
  const int r16 = lane & 15, g = lane >> 4;

  // work id: consecutive ids on one XCD (dispatch goes round-robin over XCDs);
  // tiles in groups of `group` M tiles by all N tiles, splits outermost
  const int total = (int)gridDim.x, xcd = (int)blockIdx.x % kXcds, local = (int)blockIdx.x / kXcds;
  const int per = total / kXcds, rem = total % kXcds;
  const int wid = xcd < rem ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
  const int tiles = a.tiles_m * a.tiles_n, tile = wid % tiles, split = wid / tiles;
  const int gi = tile / (a.group * a.tiles_n), gr = min(a.group, a.tiles_m - gi * a.group);
  const int gl = tile - gi * a.group * a.tiles_n;
  const int tm = gi * a.group + gl % gr, tn = gl / gr;
  const int m0 = tm * BM, n0 = tn * BN;
  const int kb0 = split * a.kbps;
  const int nkb = min(a.kbps, a.kblocks - kb0);
  const int rot = MODE == kStream ? (tile * 3) % nkb : 0;  // the K block this tile starts with

  // Copy r of this wave fills 1 KB piece p = kWaves r + w of a stage: pieces
  // below BM / 8 hold x rows 8p..8p+7, the rest W rows; lane i fetches the
  // chunk that belongs at its LDS slot (row 8p + i / 8, slot i % 8).  The piece
  // of x row M - 1 repeats that row past M, and pieces past M read that piece.
  const uint32_t lrow = lane >> 3, chunk = ((lane & 7) ^ (lane >> 3)) * 16;
  const uint32_t lrow_end = min(lrow, (uint32_t)(a.m - 1) & 7);
  const char* src[LOADS];
  uint32_t off[LOADS];
#pragma unroll
  for (int r = 0; r < LOADS; ++r) {
    const int p = r * C::kWaves + w;
    const bool isx = p < BM / 8;
    const int row0 = isx ? m0 + p * 8 : n0 + p * 8 - BM;
    const bool full = !isx || row0 + 8 <= a.m;
    const int row = full ? row0 : (a.m - 1) & ~7;
    src[r] = reinterpret_cast<const char*>(isx ? a.x : a.w) + ((size_t)row * a.k + (size_t)kb0 * BK) * 2;
    if (MODE == kWide) {
      src[r] += (size_t)(full ? lrow : lrow_end) * a.k * 2 + chunk;
      off[r] = 0;
    } else {
      off[r] = (full ? lrow : lrow_end) * (uint32_t)a.k * 2 + chunk;
    }
  }
  auto copy = [&](int r, size_t koff, const char* dst) {
    const uint32_t l = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)dst;
    if (MODE == kWide)
      dma16(src[r] + koff, dst);
    else if (MODE == kStream && r * C::kWaves + w >= BM / 8)
      asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(off[r]),
                   "s"(src[r] + koff), "{m0}"(l)
                   : "memory");
    else
      asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off[r]),
                   "s"(src[r] + koff), "{m0}"(l)
                   : "memory");
  };
  auto block_off = [&](int i) {  // byte offset of the tile's i-th K block along a row
    int kb = i + rot;
    kb = kb >= nkb ? kb - nkb : kb;
    return (size_t)kb * (BK * 2);
  };

  // fragment reads: row r16 of a 16-row tile, logical chunk 4 half + g
  const int xoff = (wm * TM * 16 + r16) * 128;
  const int woff = BM * 128 + (wn * TN * 16 + r16) * 128;
  const int c0 = (g ^ (r16 & 7)) << 4, c1 = ((4 + g) ^ (r16 & 7)) << 4;

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  // Fragments of the two halves.  kRoll: x rows 0 .. TM - 3 share one register
  // set (row t of the next half is read once row t's MFMAs are issued), the
  // last two rows have two, so their reads go out before the barrier nears.
  bf16x8 xf[2][TM], wf[2][TN];
  auto xr = [&](int b, int t) -> bf16x8& { return C::kRoll && t < TM - 2 ? xf[0][t] : xf[b][t]; };
  auto read_x = [&](int b, const char* p, int t) { xr(b, t) = as_bf16x8(ld16(p + xoff + t * 2048)); };
  auto read_w = [&](int b, const char* p, int t) { wf[b][t] = as_bf16x8(ld16(p + woff + t * 2048)); };

  int st = 0;  // stage of the current block
  // MFMAs of half b, a row of TN at a time; between the rows the fragments of
  // the other half are read from p and, with `fill`, block i's copies go out to
  // stage st.
  auto half = [&](int b, const char* p, bool fill, int i) {
    const size_t koff = fill ? block_off(i) : 0;
    const char* dst = lds + st * C::kStage + w * 1024;
#pragma unroll
    for (int t = 0; t < TM; ++t) {
#pragma unroll
      for (int nt = 0; nt < TN; ++nt) acc[t][nt] = mfma(wf[b][nt], xr(b, t), acc[t][nt]);
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (C::kRoll) {
        if (t < TM - 2) {
          read_x(b ^ 1, p, t);
#pragma unroll
          for (int j = t * TN / (TM - 2); j < (t + 1) * TN / (TM - 2); ++j) read_w(b ^ 1, p, j);
          if (t >= TM - 4) read_x(b ^ 1, p, t + 2);
        }
      } else {
        constexpr int PER = (TM + TN + TM - 1) / TM;
#pragma unroll
        for (int j = t * PER; j < (t + 1) * PER; ++j)
          if (j < TN) read_w(b ^ 1, p, j);
          else if (j < TN + TM) read_x(b ^ 1, p, j - TN);
      }
      if (fill && t * LOADS / TM < (t + 1) * LOADS / TM) {
#pragma unroll
        for (int r = t * LOADS / TM; r < (t + 1) * LOADS / TM; ++r)
          copy(r, koff, dst + r * C::kWaves * 1024);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

#pragma unroll
  for (int i = 0; i < STAGES; ++i)
    if (i < nkb) {
      const size_t koff = block_off(i);
#pragma unroll
      for (int r = 0; r < LOADS; ++r)
        copy(r, koff, lds + i * C::kStage + (r * C::kWaves + w) * 1024);
    }
  wait_blocks<STAGES - 1, LOADS>(nkb - 1);
  block_barrier();
#pragma unroll
  for (int t = 0; t < TN; ++t) read_w(0, lds + c0, t);
#pragma unroll
  for (int t = 0; t < TM; ++t) read_x(0, lds + c0, t);
  for (int i = 0; i < nkb; ++i) {
    const int next = st + 1 == STAGES ? 0 : st + 1;
    half(0, lds + st * C::kStage + c1, false, 0);
    // block i + 1 has landed (this wave's copies, then everyone's), and every
    // wave has read all of block i: its stage takes block i + STAGES.  Past the
    // last block the reads return an older block's fragments, which go unused.
    wait_blocks<STAGES - 2, LOADS>(nkb - 2 - i);
    block_barrier();
    half(1, lds + next * C::kStage + c0, i + STAGES < nkb, i + STAGES);
    st = next;
  }

  // 16-token tiles of this wave that hold rows < M (wave-uniform)
  const int nmt = max(0, min(TM, (a.m - (m0 + wm * TM * 16) + 15) / 16));
  if (a.splits > 1) {
    int& s_last = *reinterpret_cast<int*>(lds);
    float* const parts = a.part + (size_t)tile * a.splits * C::kTileFloats;
    const int mine = w * (TM * TN * 256) + lane * 4;
    const PartWriter wr(parts + (size_t)split * C::kTileFloats);
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
      if (mt < nmt)
#pragma unroll
        for (int nt = 0; nt < TN; ++nt)
          wr((mine + (mt * TN + nt) * 256) * 4, __builtin_bit_cast(u32x4, acc[mt][nt]));
    vm_wait<0>();     // this thread's device-scope stores have completed
    __syncthreads();  // everyone's have, and the ring is free
    // the tile's counter: tile % 64 names the word, tile / 64 the nibble; up to 64
    // tiles have a whole word each
    uint32_t* const word = a.tickets + tile % kTicketWords;
    const int shift = tile / kTicketWords * 4;
    const uint32_t mask = tiles <= kTicketWords ? ~0u : 15u;
    if (tid == 0) {
      const uint32_t prev =
          __hip_atomic_fetch_add(word, 1u << shift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_last = (int)((prev >> shift) & mask) == a.splits - 1;
    }
    __syncthreads();
    if (!s_last) return;
    // sum in split order, own split from registers (the same bits it stored);
    // the partials of four splits are in flight at once
    const PartReader rd(parts);
#pragma unroll
    for (int mt = 0; mt < TM; ++mt) {
      if (mt >= nmt) continue;
      f32x4 tot[TN];
#pragma unroll
      for (int nt = 0; nt < TN; ++nt) tot[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
      for (int s0 = 0; s0 < a.splits; s0 += 4) {
        f32x4 v[4][TN];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int s = s0 + j;
#pragma unroll
          for (int nt = 0; nt < TN; ++nt)
            v[j][nt] = (s < a.splits && s != split)
                           ? rd((s * C::kTileFloats + mine + (mt * TN + nt) * 256) * 4)
                           : acc[mt][nt];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (s0 + j < a.splits)
#pragma unroll
            for (int nt = 0; nt < TN; ++nt) tot[nt] += v[j][nt];
      }
#pragma unroll
      for (int nt = 0; nt < TN; ++nt) acc[mt][nt] = tot[nt];
    }
    if (tid == 0)
      __hip_atomic_fetch_sub(word, (uint32_t)a.splits << shift, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
  }

  // epilogue: lane holds n = nbase + 4 g .. + 3 of token m0 + wm TM 16 + 16 mt + r16
#pragma unroll
  for (int mt = 0; mt < TM; ++mt) {
    if (mt >= nmt) continue;
    const int tok = m0 + wm * TM * 16 + mt * 16 + r16;
    if (tok >= a.m) continue;
    const int nbase = n0 + wn * TN * 16;
    if (EPI == SSA_EPILOGUE_SWIGLU) {
      // W rows in 16-row blocks, gate block then up block of the same 16 outputs
      const int nout = a.n / 2;
#pragma unroll
      for (int j = 0; j < TN / 2; ++j) {
        const f32x4 gt = acc[mt][2 * j], up = acc[mt][2 * j + 1];
        const int col = nbase / 2 + j * 16 + g * 4;
        u32x2 v = {pack2(silu(gt[0]) * up[0], silu(gt[1]) * up[1]),
                   pack2(silu(gt[2]) * up[2], silu(gt[3]) * up[3])};
        *reinterpret_cast<u32x2*>(a.out + (size_t)tok * nout + col) = v;
      }
    } else {
#pragma unroll
      for (int nt = 0; nt < TN; ++nt) {
        const int col = nbase + nt * 16 + g * 4;
        f32x4 v = acc[mt][nt];
        if (EPI == SSA_EPILOGUE_RESIDUAL) {
          const u32x2 r = *reinterpret_cast<const u32x2*>(a.res + (size_t)tok * a.n + col);
          v[0] += bf16_lo(r[0]);
          v[1] += bf16_hi(r[0]);
          v[2] += bf16_lo(r[1]);
          v[3] += bf16_hi(r[1]);
        }
        *reinterpret_cast<u32x2*>(a.out + (size_t)tok * a.n + col) =
            u32x2{pack2(v[0], v[1]), pack2(v[2], v[3])};
      }
    }
  }
}

// RMSNorm: one workgroup per row, up to 4 16-byte chunks per thread.  `clear`:
// words that the launches behind it on the stream need to be zero (a layer's
// split tickets), spread over all threads.
constexpr int kNormChunks = 4;
__global__ __launch_bounds__(kNormThreads) void rms_norm_kernel(const uint16_t* x, const uint16_t* wt,
                                                            uint16_t* out, int n, float eps,
                                                            ssa::ClearWords clear) {
  __shared__ float s_part[kNormThreads / 64];
  const int tid = threadIdx.x;
#pragma unroll
  for (int c = 0; c < 2; ++c)
    for (int64_t i = (int64_t)blockIdx.x * kNormThreads + tid; i < clear.n[c];
         i += (int64_t)gridDim.x * kNormThreads)
      clear.at[c][i] = 0;
  const uint16_t* row = x + (size_t)blockIdx.x * n;
  u32x4 v[kNormChunks];
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < kNormChunks; ++c) {
    const int e = (c * kNormThreads + tid) * 8;
    v[c] = e < n ? ld16(row + e) : u32x4{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float lo = bf16_lo(v[c][j]), hi = bf16_hi(v[c][j]);
      ss += lo * lo + hi * hi;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
  if ((tid & 63) == 0) s_part[tid >> 6] = ss;
  __syncthreads();
  const float tot = s_part[0] + s_part[1] + s_part[2] + s_part[3];
  const float rs = __builtin_amdgcn_rsqf(tot / (float)n + eps);
#pragma unroll
  for (int c = 0; c < kNormChunks; ++c) {
    const int e = (c * kNormThreads + tid) * 8;
    if (e >= n) continue;
    const u32x4 wv = ld16(wt + e);
    u32x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      o[j] = pack2(bf16_lo(v[c][j]) * rs * bf16_lo(wv[j]), bf16_hi(v[c][j]) * rs * bf16_hi(wv[j]));
    *reinterpret_cast<u32x4*>(out + (size_t)blockIdx.x * n + e) = o;
  }
}

// The tile configurations the host chooses from, by tokens x output features.
using Cfg32x64 = TileCfg<2, 2, 1, 2, 6, 2>;
using Cfg64x64 = TileCfg<2, 2, 2, 2, 5, 2>;
using Cfg64x128 = TileCfg<2, 2, 2, 4, 3, 2>;
using Cfg96x64 = TileCfg<2, 2, 3, 2, 5, 1>;
using Cfg96x128 = TileCfg<2, 2, 3, 4, 5, 1>;
using Cfg128x64 = TileCfg<2, 2, 4, 2, 6, 1>;
using Cfg128x128 = TileCfg<2, 4, 4, 2, 5, 1>;
using Cfg160x128 = TileCfg<2, 2, 5, 4, 2, 2>;
using Cfg192x128 = TileCfg<4, 2, 3, 4, 4, 1>;
using Cfg192x128x2 = TileCfg<2, 2, 6, 4, 2, 2>;
using Cfg256x128 = TileCfg<4, 2, 4, 4, 3, 1>;
using Cfg256x256 = TileCfg<2, 4, 8, 4, 2, 1>;
enum {
  kCfg32x64, kCfg64x64, kCfg64x128, kCfg96x64, kCfg96x128, kCfg128x64, kCfg128x128,
  kCfg160x128, kCfg192x128, kCfg192x128x2, kCfg256x128, kCfg256x256, kNumCfgs
};

struct CfgShape {
  int bm, bn, occ, stages, threads;
};
template <class C>
constexpr CfgShape shape_of() {
  return CfgShape{C::BM, C::BN, C::OCC, C::STAGES, C::kThreads};
}
constexpr CfgShape kCfgShapes[kNumCfgs] = {
    shape_of<Cfg32x64>(),   shape_of<Cfg64x64>(),   shape_of<Cfg64x128>(),    shape_of<Cfg96x64>(),
    shape_of<Cfg96x128>(),  shape_of<Cfg128x64>(),  shape_of<Cfg128x128>(),   shape_of<Cfg160x128>(),
    shape_of<Cfg192x128>(), shape_of<Cfg192x128x2>(), shape_of<Cfg256x128>(), shape_of<Cfg256x256>()};

struct GemmPlan {
  int cfg, tiles_m, tiles_n, splits, kbps, kblocks;
  size_t ws;
};

constexpr int kCus = 256;
// Split tickets: a counter per tile in the workspace's first 256 bytes, whatever
// the shape, so that products of different shapes can share a workspace (the
// partials of one never lie where another's tickets are): a word each for up to
// 64 tiles, else 4 bits.
constexpr int kMaxSplitTiles = kTicketWords * 8;
constexpr int max_splits(int64_t tiles) { return tiles <= kTicketWords ? 256 : 15; }

// cfg's tiles in (up to) s K splits; one where the tickets do not suffice.
GemmPlan make_plan(int cfg, int m, int n, int k, int s) {
  const CfgShape& cs = kCfgShapes[cfg];
  GemmPlan c;
  c.cfg = cfg;
  c.tiles_m = (m + cs.bm - 1) / cs.bm;
  c.tiles_n = n / cs.bn;
  c.kblocks = k / BK;
  const int64_t tiles = (int64_t)c.tiles_m * c.tiles_n;
  s = tiles > kMaxSplitTiles ? 1 : std::max(1, std::min({s, c.kblocks, max_splits(tiles)}));
  c.kbps = (c.kblocks + s - 1) / s;
  c.splits = (c.kblocks + c.kbps - 1) / c.kbps;
  c.ws = c.splits > 1 ? kTicketBytes + (size_t)c.tiles_m * c.tiles_n * c.splits * cs.bm * cs.bn * 4 : 0;
  return c;
}

// Microseconds a workgroup of each configuration takes per K block of 64, with
// one and (OCC 2) two of them on every CU.  Fitted, with the constants of
// plan_cost, to 290 products timed on MI355X in every configuration and 1 to 12
// splits, weights out of the caches (M = 1 .. 4096; N x K of the Llama-3-8B
// projections and 640 x 640 .. 16384 x 8192).  On 286 other products (M = 4 .. 1400,
// 2048 x 2048 .. 57344 x 8192) the plan picked takes 1.01 of the time of the fastest
// plan on the mean and 1.23 at worst; on the Llama-3-8B projections 0.69 of
// hipBLASLt's time for M <= 256, 0.98 from 384 to 1152 and 1.12 from 2176 on.
constexpr double kBlockUs[kNumCfgs][2] = {
    {0.182, 0.293}, {0.239, 0.475}, {0.380, 0.629}, {0.281, 0.281}, {0.453, 0.453}, {0.379, 0.379},
    {0.521, 0.521}, {0.832, 1.126}, {0.662, 0.662}, {0.924, 1.278}, {0.827, 0.827}, {1.447, 1.447}};

// Estimated microseconds of a plan: rounds of the chip's workgroup slots times
// a workgroup's K blocks (its pipeline's fill counted as 1.3 more; a last round
// of the tall tiles that come two to a CU costs by the CUs that hold two, an only
// round at least 0.6 of the way to all of them: 377 x 18432 x 7168 in 288 workgroups
// took 159 us, 126 in 432), or the weights' bytes, whichever is larger; and for a
// split the last arriver's reads of the other partial tiles and all their bytes.
// The bytes move at less where the workgroups' copies in flight are too few to
// hide the latency, and, with one M tile of few rows, where some CUs hold a
// workgroup more than others (8 x 10240 x 8192 in 320 workgroups 35 us, in 160 or
// 480 30 us).
double plan_cost(const GemmPlan& c, int m, int n, int k) {
  const CfgShape& cs = kCfgShapes[c.cfg];
  const double one = kBlockUs[c.cfg][0], two = kBlockUs[c.cfg][1];
  const int64_t wgs = (int64_t)c.tiles_m * c.tiles_n * c.splits, slots = (int64_t)kCus * cs.occ;
  const int64_t rest = wgs % slots;
  double t = (double)(wgs / slots) * two;
  const double paired = std::max((double)(rest - kCus) / kCus, wgs < slots ? 0.6 : 0.);
  if (rest > kCus) t += cs.bm >= 160 ? one + (two - one) * paired : two;
  else if (rest > 0) t += one;
  t *= c.kbps + 1.3;
  const double in_flight = (double)wgs * cs.bn * (cs.stages - 1) / 64.;
  double uneven = 1.;
  if (c.tiles_m == 1 && cs.bm <= 64 && wgs > kCus)
    uneven += 0.4 * ((double)((wgs + kCus - 1) / kCus * kCus) / wgs - 1.);
  t = std::max(t, (double)n * k * 2. / 8.59e6 / std::min(1., in_flight / 1016.) * uneven);
  if (c.splits > 1) {
    const double tile = (double)std::min(cs.bm, (m + 15) / 16 * 16) * cs.bn;
    t += 3.41 + (c.splits - 1) * tile * (1.545 / 16384.);
    t += (double)c.tiles_m * c.tiles_n * (c.splits - 1) * tile * 4. / 2.325e6;
  }
  return t;
}

// A launch holds fewer than 2^32 threads.
bool launchable(const GemmPlan& c) {
  return (int64_t)c.tiles_m * c.tiles_n * c.splits * kCfgShapes[c.cfg].threads < INT64_C(1) << 32;
}

// The cheapest plan by plan_cost over the configurations and 1 .. 12 splits of
// at least 3 K blocks that leave at most 1100 workgroups.  A few tiles on a long K
// (at least 32 K blocks a split, so K >= 32768) are cut further, up to 256 ways:
// 1 x 128 x 2^20 91 us, 529 in 12 splits; 16 x 128 x 65536 14 us and 23.
GemmPlan choose_plan(int m, int n, int k, int most_splits = 256) {
  GemmPlan best{};
  double best_cost = 1e300;
  const bool small_fits = launchable(make_plan(kCfg32x64, m, n, k, 1));
  for (int cfg = 0; cfg < kNumCfgs; ++cfg) {
    const CfgShape& cs = kCfgShapes[cfg];
    if (k >= kWideK && cfg != kCfg32x64) break;  // the one with 64-bit lane addresses
    // half-empty tiles, and tiles far smaller than a long batch, never win
    if (k < kWideK && (n % cs.bn || (small_fits && cs.bm > 32 && cs.bm >= 2 * m) ||
                       (cs.bm < 96 && m >= 1024)))
      continue;
    // (every size that check_linear takes is launchable in 64 x 128 tiles)
    if (!launchable(make_plan(cfg, m, n, k, 1))) continue;
    for (int s : {1, 2, 3, 4, 5, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256}) {
      if (s > most_splits) break;
      const GemmPlan c = make_plan(cfg, m, n, k, s);
      if (s > 1 && ((int64_t)c.tiles_m * c.tiles_n * s > 1100 || c.kblocks / s < 3)) break;
      if (s > 12 && (s > max_splits((int64_t)c.tiles_m * c.tiles_n) || c.kblocks / s < 32)) break;
      const double cost = plan_cost(c, m, n, k);
      if (cost < best_cost) best_cost = cost, best = c;
    }
  }
  return best;
}

// Products that run without a workspace too, in one pass over K: those whose tiles
// of 64 x 128 give half of the CUs one (a quarter of them up to 64 tokens, where
// the weights' bytes bound it).  The splits they have with a workspace gain up to a
// fifth, or nothing: 39 x 10240 x 6528 26.6 us, 32.3 without; 1600 x 4096 x 14336
// 168 and 175; 391 x 8832 x 7872 72 and 72.
bool runs_unsplit(int m, int n) {
  return (int64_t)((m + 63) / 64) * (n / 128) >= (m <= 64 ? kCus / 4 : kCus / 2);
}

template <class C, int MODE>
void launch_mode(const GemmPlan& c, int epilogue, const GemmArgs& a, hipStream_t s) {
  const dim3 grid(c.tiles_m * c.tiles_n * c.splits), block(C::kThreads);
  if (epilogue == SSA_EPILOGUE_NONE)
    hipLaunchKernelGGL((linear_kernel<C, SSA_EPILOGUE_NONE, MODE>), grid, block, 0, s, a);
  else if (epilogue == SSA_EPILOGUE_RESIDUAL)
    hipLaunchKernelGGL((linear_kernel<C, SSA_EPILOGUE_RESIDUAL, MODE>), grid, block, 0, s, a);
  else
    hipLaunchKernelGGL((linear_kernel<C, SSA_EPILOGUE_SWIGLU, MODE>), grid, block, 0, s, a);
}

template <class C>
void launch_cfg(const GemmPlan& c, int epilogue, const GemmArgs& a, hipStream_t s) {
  if (c.tiles_m == 1) launch_mode<C, kStream>(c, epilogue, a, s);
  else launch_mode<C, kShared>(c, epilogue, a, s);
}

// Launch a planned product; the workspace has been checked against c.ws.
int launch_linear(const GemmPlan& c, int m, int n, int k, int epilogue, const uint16_t* x,
                  const uint16_t* w, const uint16_t* residual, uint16_t* out, void* workspace,
                  hipStream_t s) {
  GemmArgs a{x, w, residual, out,
             static_cast<uint32_t*>(workspace),
             c.ws > 0 ? reinterpret_cast<float*>(static_cast<char*>(workspace) + kTicketBytes) : nullptr,
             m, n, k, c.tiles_m, c.tiles_n, c.splits, c.kbps, c.kblocks,
             // up to 8 M tiles: all of them beside each N tile; more: groups of 4
             c.tiles_m <= 8 ? c.tiles_m : 4};
  (void)hipGetLastError();
  switch (c.cfg) {
    case kCfg32x64:
      if (k >= kWideK) launch_mode<Cfg32x64, kWide>(c, epilogue, a, s);
      else launch_cfg<Cfg32x64>(c, epilogue, a, s);
      break;
    case kCfg64x64: launch_cfg<Cfg64x64>(c, epilogue, a, s); break;
    case kCfg64x128: launch_cfg<Cfg64x128>(c, epilogue, a, s); break;
    case kCfg96x64: launch_cfg<Cfg96x64>(c, epilogue, a, s); break;
    case kCfg96x128: launch_cfg<Cfg96x128>(c, epilogue, a, s); break;
    case kCfg128x64: launch_cfg<Cfg128x64>(c, epilogue, a, s); break;
    case kCfg128x128: launch_cfg<Cfg128x128>(c, epilogue, a, s); break;
    case kCfg160x128: launch_cfg<Cfg160x128>(c, epilogue, a, s); break;
    case kCfg192x128: launch_cfg<Cfg192x128>(c, epilogue, a, s); break;
    case kCfg192x128x2: launch_cfg<Cfg192x128x2>(c, epilogue, a, s); break;
    case kCfg256x128: launch_cfg<Cfg256x128>(c, epilogue, a, s); break;
    default: launch_cfg<Cfg256x256>(c, epilogue, a, s); break;
  }
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

// Sizes whose tile counts fit the plan's 32-bit fields (at most 2^25 of the
// smallest tile, 32 x 64; only up to 512 tiles are split), which some
// configuration's grid can hold, and whose operands stay below 2^40 elements.
int check_linear(int32_t m, int32_t n, int32_t k, int32_t epilogue) {
  if (m < 0 || n <= 0 || k <= 0 || n % 128 || k % BK) return SSA_ERR_ARG;
  if (epilogue < SSA_EPILOGUE_NONE || epilogue > SSA_EPILOGUE_SWIGLU) return SSA_ERR_ARG;
  if ((int64_t)m * k > INT64_C(1) << 40 || (int64_t)n * k > INT64_C(1) << 40) return SSA_ERR_ARG;
  if ((int64_t)(m / 32 + 1) * (n / 128) > INT64_C(1) << 24) return SSA_ERR_ARG;
  return SSA_OK;
}

}  // namespace

namespace ssa {

int rms_norm(int32_t m, int32_t n, const uint16_t* x, const uint16_t* weight, float eps,
             uint16_t* out, const ClearWords& clear, void* stream) {
  if (m < 0 || n <= 0 || n % 8 || n > kNormThreads * 8 * kNormChunks || !(eps >= 0.f))
    return SSA_ERR_ARG;
  if (m == 0) return SSA_OK;
  if (!x || !weight || !out) return SSA_ERR_NULL;
  (void)hipGetLastError();
  hipLaunchKernelGGL(rms_norm_kernel, dim3(m), dim3(kNormThreads), 0, static_cast<hipStream_t>(stream),
                     x, weight, out, n, eps, clear);
  return hipGetLastError() == hipSuccess ? SSA_OK : SSA_ERR_HIP;
}

}  // namespace ssa

extern "C" {

int ssa_linear_workspace_size(int32_t m, int32_t n, int32_t k, size_t* ws_bytes) {
  if (!ws_bytes) return SSA_ERR_NULL;
  const int rc = check_linear(m, n, k, SSA_EPILOGUE_NONE);
  if (rc) return rc;
  *ws_bytes = m == 0 ? 0 : choose_plan(m, n, k).ws;
  return SSA_OK;
}

int ssa_linear_plan(int32_t m, int32_t n, int32_t k, ssa_linear_plan_info* info) {
  if (!info) return SSA_ERR_NULL;
  const int rc = check_linear(m, n, k, SSA_EPILOGUE_NONE);
  if (rc) return rc;
  *info = ssa_linear_plan_info{};
  if (m == 0) return SSA_OK;
  const GemmPlan c = choose_plan(m, n, k);
  const CfgShape& cs = kCfgShapes[c.cfg];
  *info = ssa_linear_plan_info{cs.bm, cs.bn, cs.threads, c.tiles_m, c.tiles_n, c.splits};
  return SSA_OK;
}

int ssa_linear(int32_t m, int32_t n, int32_t k, int32_t epilogue, const uint16_t* x,
               const uint16_t* w, const uint16_t* residual, uint16_t* out, void* workspace,
               size_t ws_bytes, void* stream) {
  const int rc = check_linear(m, n, k, epilogue);
  if (rc) return rc;
  if (m == 0) return SSA_OK;
  if (!x || !w || !out || (epilogue == SSA_EPILOGUE_RESIDUAL && !residual)) return SSA_ERR_NULL;
  GemmPlan c = choose_plan(m, n, k);
  if (c.ws > 0 && (!workspace || ws_bytes < c.ws)) {
    if (!runs_unsplit(m, n)) return SSA_ERR_WORKSPACE;
    c = choose_plan(m, n, k, 1);
  }
  return launch_linear(c, m, n, k, epilogue, x, w, residual, out, workspace,
                       static_cast<hipStream_t>(stream));
}

int ssa_rms_norm(int32_t m, int32_t n, const uint16_t* x, const uint16_t* weight, float eps,
                 uint16_t* out, void* stream) {
  return ssa::rms_norm(m, n, x, weight, eps, out, ssa::ClearWords{}, stream);
}

}  // extern "C"
