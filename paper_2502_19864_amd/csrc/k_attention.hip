// Attention core of the frozen blocks: softmax(Q K^T / sqrt(d_head) [+causal]) V
// per (batch, head), and its backward (dQ, dK, dV; frozen projections around it
// are plain GEMMs).  Rotary embedding (rotate-half pairs (i, i + d_head/2)):
// in bf16 stages the QKV projection's epilogue has already rotated Q and K, so
// the stash holds the rotated projections and the kernels load them as they
// are.  The backward rotates dQ and dK back before storing them.
//
// bf16 kernels use MFMA 32x32x16 with K/V (or Q/dO) tiles staged in LDS.
// Each wave owns 32 queries (forward, dQ pass) or 32 keys (dK/dV pass), so the
// score block held in registers has a fixed query (key) per lane and the
// softmax row statistics are mostly in-lane.  The probabilities are fed back
// to the second MFMA straight from registers: within one 16-wide k step the
// lane's values cover 16 keys in a fixed permuted order, and the other operand
// is read in that same order from the row-major LDS tile with the gfx950 LDS
// transpose read (ds_read_b64_tr_b16), so no tile is ever stored transposed.
//
// Log-sum-exp is kept in base 2 of the scaled scores: lse2 = log2 sum_j
// 2^(s_j * scale * log2 e).
#include "attn_core.h"
#include "common.h"
#include "kernels.h"

namespace rg {

// ================================================================ bf16 / MFMA
// One [KT x DH] tile of rows r0.. (rows >= S are zero) from column col of a
// row-major source into LDS row-major (pitch DH + 8), in two steps so that the
// caller can issue the global loads of several tiles before the first LDS
// store: issue() loads this thread's 16-B chunks into registers, store()
// writes them.
template <int DH, int NT>
struct TileLoad {
  static constexpr int HC = DH / 16, PAIRS = KT * HC, IT = PAIRS / NT;
  static_assert(PAIRS % NT == 0, "whole passes of the workgroup");
  bf16x8 raw[IT][2];
  __device__ __forceinline__ void issue(const bf16* src, int ld, int col, int b, int S, int r0) {
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int p = threadIdx.x + it * NT;
      // rows past S read row S - 1 and are zeroed in store(): no load is conditional on
      // a lane, so none waits for the one before it
      const int r = p / HC, c = p % HC, row = min(r0 + r, S - 1);
      const bf16* a0 = src + (long)(b * S + row) * ld + col + c * 8;
      raw[it][0] = ld_frag(a0);
      raw[it][1] = ld_frag(a0 + DH / 2);
    }
  }
  __device__ __forceinline__ void store(bf16* dst, int S, int r0) {
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int p = threadIdx.x + it * NT;
      const int r = p / HC, c = p % HC, row = r0 + r;
      if (row >= S) raw[it][0] = raw[it][1] = zero_frag();
      *reinterpret_cast<bf16x8*>(dst + r * (DH + 8) + c * 8) = raw[it][0];
      *reinterpret_cast<bf16x8*>(dst + r * (DH + 8) + c * 8 + DH / 2) = raw[it][1];
    }
  }
};

// Fragments (B operand, k = head dim) of one row held by this lane: dims
// 16s + 8*(lane/32) + v, zero when !valid (src is a valid row even then: the loads are
// unconditional and issued together, the values masked afterwards).
template <int DH>
__device__ __forceinline__ void load_row_frags(const bf16* src, bool valid, int half, bf16x8 f[DH / 16]) {
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) f[s] = ld_frag(src + 16 * s + 8 * half);
#pragma unroll
  for (int s = 0; s < DH / 16; ++s)
    if (!valid) f[s] = zero_frag();
}

// ---------------------------------------------------------------- tiles by DMA
// A [R x DH] tile goes global -> LDS by DMA, rows unpadded (the DMA writes 1 KB runs):
// 16-B chunk c of row r sits at c ^ swz(r).  The swizzle has to serve two reads:
// ld_frag of one chunk of 16 consecutive rows (all sixteen must land on
// different 16-B slots of the 256 B that one pass of the LDS covers), and the
// transpose read of four chunks of four consecutive rows (each row on a 64-B
// group of its own; rows padded by 16 B, as before, put all four on two groups).
template <int DH>
__device__ __forceinline__ int swz(int r) {
  return DH == 128 ? ((r & 3) << 2) | ((r >> 2) & 3) : (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
}
// rows r0 .. r0 + R - 1 (r0 < S; rows past S - 1 read that row: their scores are masked)
// of column col; the caller waits with tiles_ready
template <int DH, int R, int NW>
__device__ __forceinline__ void tile_dma(const bf16* src, int ld, int col, int b, int S, int r0, bf16* dst) {
  constexpr int CPR = DH / 8, RPI = 64 / CPR;
  static_assert(R % (RPI * NW) == 0, "whole DMA instructions per wave");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bf16* base = src + ((long)b * S + r0) * ld + col;
#pragma unroll
  for (int i = 0; i < R / (RPI * NW); ++i) {
    const int r = (i * NW + wave) * RPI + lane / CPR, c = (lane % CPR) ^ swz<DH>(r);
    dma16_m0(base, (uint32_t)((min(r, S - 1 - r0) * ld + c * 8) * 2), lds_addr(dst) + (i * NW + wave) * 1024);
  }
}
// this wave's DMAs have landed and its LDS reads are done, then everybody's
__device__ __forceinline__ void tiles_ready() {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}
// Element offsets of this lane's reads in such a tile: row for dims 8*half of row
// lane%32, tr for perm_frag's transpose read of block 0.  The swizzle is an XOR
// below the row bits, so other dims are reached by an XOR of their own (16s, 32
// db) and the rows 8 further down, whose swizzle differs in bit 1 of the chunk, by 16;
// rows + 16 i are constant offsets.
template <int DH>
struct TileRead {
  int row, tr;
  __device__ __forceinline__ explicit TileRead(int lane) {
    const int l32 = lane & 31, half = lane >> 5, g = lane >> 4, r = lane & 15;
    row = l32 * DH + ((half ^ swz<DH>(l32)) * 8);
    const int rr = 4 * (g >> 1) + (r >> 2), c = 2 * (g & 1) + ((r & 3) >> 1);
    tr = rr * DH + ((c ^ swz<DH>(rr)) * 8) + 4 * (r & 1);
  }
  // fragment of rows kb*32 + lane%32, dims 16s + 8*half + 0..7
  __device__ __forceinline__ bf16x8 frag(const bf16* tile, int kb, int s) const {
    return ld_frag(tile + (row ^ (16 * s)) + kb * 32 * DH);
  }
  // the same operand as perm_frag
  __device__ __forceinline__ bf16x8 perm(const bf16* tile, int db, int kb, int j) const {
    const bf16* lo = tile + (tr ^ (32 * db)) + (kb * 32 + 16 * j) * DH;
    const bf16* hi = tile + (tr ^ (32 * db) ^ 16) + (kb * 32 + 16 * j + 8) * DH;
    const uint2 l = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)lo));
    const uint2 h = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16_ptr)hi));
    return __builtin_bit_cast(bf16x8, make_uint4(l.x, l.y, h.x, h.y));
  }
};

// Causal tiles do unequal work: query tile t of nq takes t + 1 key tiles (the dK/dV
// pass: key block j takes nq - j query tiles).  At d_h = 128 a workgroup fills its CU,
// so the CUs take the workgroups in dispatch order as they free up; dispatching the
// heaviest tiles first (each XCD gets its workgroups in linear-id order, one in eight)
// keeps the light ones for the end, where the plain order could leave one CU a heavy
// tile last.  Returns rank 0 for the heaviest tile and the batch-head index; shapes
// whose workgroups do not split evenly over the XCDs keep xcd_block's order.
__device__ __forceinline__ void heavy_first(int lin, int nq, int nbh, int& rank, int& bh) {
  const int n = nq * nbh, P = n / 8;
  if (n % 8 || P % nq) {
    const int blk = xcd_block(lin, n);
    rank = nq - 1 - blk % nq;
    bh = blk / nq;
    return;
  }
  const int x = lin % 8, o = lin / 8, per = P / nq;  // XCD x, its o-th workgroup
  rank = o / per;
  bh = x * per + o % per;
}

// Forward and the two backward passes for more than one tile.  Each works
// through tiles of KR rows of the other side, two deep in LDS by DMA (one barrier
// per tile, no registers held for the loads), and skips, wave by wave, blocks
// that the causal mask or the sequence's end leaves empty.  KR 64 and no staging
// registers keep d_head 128 within two waves per SIMD (one before: nothing
// overlapped the softmax with MFMAs and LDS reads); only the dK/dV pass still
// spills there (19 registers causal, 7 not).  Results leave through LDS as whole
// rows.  The forward's running maximum moves once per 64 keys (128 before), so P is
// rounded to bf16 at other scales: other bits, the same error against 64 bits.
// Before -> after, us: 2048 tokens of 512, 32 heads of 128, causal: forward 43 -> 23,
// dQ 56 -> 40, dK/dV 71 -> 57; 4096 tokens of 256, 16 heads of 64: 15.8 -> 13.6,
// 20.4 -> 20.4, 28.6 -> 21.4.
template <int DH, bool CAUSAL, int NW, int KR>
__global__ __launch_bounds__(64 * NW, 2) void attn_fwd_bf16(AttnArgs a) {
  constexpr int TILE = KR * DH;
  __shared__ __attribute__((aligned(1024))) bf16 sm[4 * TILE];  // [buffer][K, V]
  static_assert(4 * TILE >= NW * 32 * (DH + 8), "the O rows fit the tiles' space");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, l32 = lane & 31;
  int qb, bh;
  if (CAUSAL) {
    heavy_first(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x, gridDim.y, qb, bh);
    qb = gridDim.x - 1 - qb;  // query tile t does t + 1 key tiles
  } else {
    const int blk = xcd_block(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
    qb = blk % gridDim.x;
    bh = blk / gridDim.x;
  }
  const int b = bh / a.H, hd = bh % a.H, S = a.S;
  const int q0 = qb * (32 * NW) + wave * 32, q = q0 + l32;  // this wave's first query, this lane's
  const bool qv = q < S;
  const float sl2 = kLog2e * rsqrtf((float)DH);
  const bf16* qkv = static_cast<const bf16*>(a.qkv);
  const TileRead<DH> rd(lane);
  auto issue = [&](int kt) {
    bf16* dst = sm + (kt & 1) * 2 * TILE;
    tile_dma<DH, KR, NW>(qkv, a.ld_qkv, a.qkv_ko + hd * a.qkv_hs, b, S, kt * KR, dst);
    tile_dma<DH, KR, NW>(qkv, a.ld_qkv, a.qkv_vo + hd * a.qkv_hs, b, S, kt * KR, dst + TILE);
  };
  issue(0);
  bf16x8 qf[DH / 16];
  load_row_frags<DH>(qkv + (long)(b * S + (qv ? q : 0)) * a.ld_qkv + hd * a.qkv_hs, qv, half, qf);

  f32x16 oacc[DH / 32];
#pragma unroll
  for (int i = 0; i < DH / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[i][r] = 0.f;
  float mrun = -INFINITY, lrun = 0.f;

  const int qlast = min(S - 1, qb * (32 * NW) + 32 * NW - 1);
  const int nkt = CAUSAL ? qlast / KR + 1 : (S + KR - 1) / KR;
  for (int kt = 0; kt < nkt; ++kt) {
    tiles_ready();
    if (kt + 1 < nkt) issue(kt + 1);
    if (q0 >= S || (CAUSAL && kt * KR > q0 + 31)) continue;  // wave-uniform: nothing to do in this tile
    const bf16* sK = sm + (kt & 1) * 2 * TILE;
    const bf16* sV = sK + TILE;
    f32x16 sc[KR / 32];
#pragma unroll
    for (int kb = 0; kb < KR / 32; ++kb) {
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[kb][r] = 0.f;
#pragma unroll
      for (int s = 0; s < DH / 16; ++s) sc[kb] = mfma32(rd.frag(sK, kb, s), qf[s], sc[kb]);
    }
    // the row max on the raw scores (the scale is positive), the scale folded
    // into the exponent's FMA; masking only where a key can be out of range
    // or in the future
    float mx = -INFINITY;
    if ((CAUSAL && (kt + 1) * KR - 1 > q0) || (kt + 1) * KR > S) {
#pragma unroll
      for (int kb = 0; kb < KR / 32; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = kt * KR + kb * 32 + perm_pos(r, half);
          const bool ok = key < S && (!CAUSAL || key <= q);
          sc[kb][r] = ok ? sc[kb][r] : -INFINITY;
          mx = fmaxf(mx, sc[kb][r]);
        }
    } else {
#pragma unroll
      for (int kb = 0; kb < KR / 32; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[kb][r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float mnew = fmaxf(mrun, mx * sl2);
    const float alpha = __builtin_amdgcn_exp2f(mrun - mnew);  // 0 on the first tile
    float rs = 0.f;
#pragma unroll
    for (int kb = 0; kb < KR / 32; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sc[kb][r] = __builtin_amdgcn_exp2f(fmaf(sc[kb][r], sl2, -mnew));
        rs += sc[kb][r];
      }
    rs += __shfl_xor(rs, 32, 64);
    lrun = lrun * alpha + rs;
    mrun = mnew;
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[i][r] *= alpha;
#pragma unroll
    for (int kb = 0; kb < KR / 32; ++kb)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 pf = pack8(sc[kb], j);
#pragma unroll
        for (int db = 0; db < DH / 32; ++db) oacc[db] = mfma32(rd.perm(sV, db, kb, j), pf, oacc[db]);
      }
  }
  tiles_ready();  // the tiles' space now takes the O rows
  if (q0 >= S) return;
  store_rows_staged<DH>(oacc, 1.f / lrun, half, lane, sm + wave * 32 * (DH + 8),
                        static_cast<bf16*>(a.o) + (long)(b * S + q0) * a.ld_o + hd * DH, a.ld_o,
                        stream_out((long)a.B * S * a.H * DH * 2), S - q0);
  if (qv && half == 0) a.lse[(long)bh * S + q] = mrun + log2f(lrun);
}

// dQ pass (lane = query); also writes D = rowsum(dO * O)
template <int DH, bool CAUSAL, int NW, int KR>
__global__ __launch_bounds__(64 * NW, 2) void attn_bwd_dq_bf16(AttnArgs a) {
  constexpr int TILE = KR * DH;
  __shared__ __attribute__((aligned(1024))) bf16 sm[4 * TILE];  // [buffer][K, V]
  static_assert(4 * TILE >= NW * 32 * (DH + 8), "the dQ rows fit the tiles' space");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, l32 = lane & 31;
  int qb, bh;
  if (CAUSAL) {
    heavy_first(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x, gridDim.y, qb, bh);
    qb = gridDim.x - 1 - qb;  // query tile t does t + 1 key tiles
  } else {
    const int blk = xcd_block(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
    qb = blk % gridDim.x;
    bh = blk / gridDim.x;
  }
  const int b = bh / a.H, hd = bh % a.H, S = a.S;
  const int q0 = qb * (32 * NW) + wave * 32, q = q0 + l32;
  const bool qv = q < S;
  const float scale = rsqrtf((float)DH), sl2 = kLog2e * scale;
  const bf16* qkv = static_cast<const bf16*>(a.qkv);
  const long qrow = (long)(b * S + (qv ? q : 0));
  const TileRead<DH> rd(lane);
  auto issue = [&](int kt) {
    bf16* dst = sm + (kt & 1) * 2 * TILE;
    tile_dma<DH, KR, NW>(qkv, a.ld_qkv, a.qkv_ko + hd * a.qkv_hs, b, S, kt * KR, dst);
    tile_dma<DH, KR, NW>(qkv, a.ld_qkv, a.qkv_vo + hd * a.qkv_hs, b, S, kt * KR, dst + TILE);
  };
  issue(0);
  bf16x8 qf[DH / 16], df[DH / 16];
  load_row_frags<DH>(qkv + qrow * a.ld_qkv + hd * a.qkv_hs, qv, half, qf);
  load_row_frags<DH>(static_cast<const bf16*>(a.dout) + qrow * a.ld_do + hd * DH, qv, half, df);
  float dsum = 0.f;
  {
    bf16x8 of[DH / 16];
    load_row_frags<DH>(static_cast<const bf16*>(a.o) + qrow * a.ld_o + hd * DH, qv, half, of);
#pragma unroll
    for (int s = 0; s < DH / 16; ++s) {
      float ov[8], dv[8];
      unpack_frag(of[s], ov);
      unpack_frag(df[s], dv);
#pragma unroll
      for (int v = 0; v < 8; ++v) dsum += ov[v] * dv[v];
    }
    dsum += __shfl_xor(dsum, 32, 64);
  }
  const float lse_raw = a.lse[(long)bh * S + (qv ? q : 0)];
  const float lse = qv ? lse_raw : 0.f;
  if (qv && half == 0) a.dsum[(long)bh * S + q] = dsum;

  f32x16 dq[DH / 32];
#pragma unroll
  for (int i = 0; i < DH / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[i][r] = 0.f;

  const int qlast = min(S - 1, qb * (32 * NW) + 32 * NW - 1);
  const int nkt = CAUSAL ? qlast / KR + 1 : (S + KR - 1) / KR;
  for (int kt = 0; kt < nkt; ++kt) {
    tiles_ready();
    if (kt + 1 < nkt) issue(kt + 1);
    if (q0 >= S) continue;
    const bf16* sK = sm + (kt & 1) * 2 * TILE;
    const bf16* sV = sK + TILE;
    // one key block at a time (not unrolled): keeps the kernel within the
    // registers of two waves per SIMD
#pragma unroll 1
    for (int kb = 0; kb < KR / 32; ++kb) {
      const int k0 = kt * KR + kb * 32;
      if (k0 >= S || (CAUSAL && k0 > q0 + 31)) break;  // wave-uniform
      // every query and key of the block in range, none masked
      const bool full = q0 + 32 <= S && k0 + 32 <= S && (!CAUSAL || k0 + 31 <= q0);
      f32x16 st, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) st[r] = dp[r] = 0.f;
#pragma unroll
      for (int s = 0; s < DH / 16; ++s) {
        st = mfma32(rd.frag(sK, kb, s), qf[s], st);
        dp = mfma32(rd.frag(sV, kb, s), df[s], dp);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = k0 + perm_pos(r, half);
        const bool ok = full || (qv && key < S && (!CAUSAL || key <= q));
        const float p = ok ? __builtin_amdgcn_exp2f(fmaf(st[r], sl2, -lse)) : 0.f;
        st[r] = p * (dp[r] - dsum);  // dS
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 sf = pack8(st, j);
#pragma unroll
        for (int db = 0; db < DH / 32; ++db) dq[db] = mfma32(rd.perm(sK, db, kb, j), sf, dq[db]);
      }
    }
  }
  tiles_ready();  // the tiles' space now takes the dQ rows
  if (q0 >= S) return;
  if (a.rope) unrotate<DH>(dq, min(q, S - 1), a.rope_tab, half);
  store_rows_staged<DH>(dq, scale, half, lane, sm + wave * 32 * (DH + 8),
                        static_cast<bf16*>(a.dqkv) + (long)(b * S + q0) * a.ld_dqkv + hd * DH, a.ld_dqkv,
                        stream_out(3l * a.B * S * a.H * DH * 2), S - q0);
}

// dK/dV pass (lane = key)
template <int DH, bool CAUSAL, int NW, int KR>
__global__ __launch_bounds__(64 * NW, 2) void attn_bwd_dkdv_bf16(AttnArgs a) {
  constexpr int TILE = KR * DH;
  __shared__ __attribute__((aligned(1024))) bf16 sm[4 * TILE];  // [buffer][Q, dO]
  __shared__ __attribute__((aligned(16))) float sL[2][KR], sD[2][KR];
  static_assert(4 * TILE >= NW * 32 * (DH + 8) && KR <= 64 * NW, "the dK / dV rows fit the tiles' space");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, l32 = lane & 31;
  int kb0, bh;
  if (CAUSAL) {
    heavy_first(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x, gridDim.y, kb0, bh);  // block j: nq - j tiles
  } else {
    const int blk = xcd_block(blockIdx.x + gridDim.x * blockIdx.y, gridDim.x * gridDim.y);
    kb0 = blk % gridDim.x;
    bh = blk / gridDim.x;
  }
  const int b = bh / a.H, hd = bh % a.H, S = a.S;
  const int k0 = kb0 * (32 * NW) + wave * 32, key = k0 + l32;  // this wave's first key, this lane's
  const bool kv = key < S;
  const int d = a.H * DH;
  const float scale = rsqrtf((float)DH), sl2 = kLog2e * scale;
  const bf16* qkv = static_cast<const bf16*>(a.qkv);
  const long krow = (long)(b * S + (kv ? key : 0));
  TileRead<DH> rd(lane);
  const int nqt = (S + KR - 1) / KR, qt0 = CAUSAL ? (kb0 * (32 * NW)) / KR : 0;
  auto issue = [&](int qt) {
    bf16* dst = sm + (qt & 1) * 2 * TILE;
    tile_dma<DH, KR, NW>(qkv, a.ld_qkv, hd * a.qkv_hs, b, S, qt * KR, dst);
    tile_dma<DH, KR, NW>(static_cast<const bf16*>(a.dout), a.ld_do, hd * DH, b, S, qt * KR, dst + TILE);
  };
  // the row statistics of tile qt, one query per thread of the first KR (rows past S: 0)
  auto load_stats = [&](int qt, float& lv, float& dv) {
    const int qq = qt * KR + (int)threadIdx.x;
    const long qi = (long)bh * S + min(qq, S - 1);
    lv = dv = 0.f;
    if (threadIdx.x < KR) {
      lv = a.lse[qi];
      dv = a.dsum[qi];
      if (qq >= S) lv = dv = 0.f;
    }
  };
  auto put_stats = [&](int qt, float lv, float dv) {
    if (threadIdx.x < KR) {
      sL[qt & 1][threadIdx.x] = lv;
      sD[qt & 1][threadIdx.x] = dv;
    }
  };
  issue(qt0);
  float lnext, dnext;
  load_stats(qt0, lnext, dnext);
  bf16x8 kf[DH / 16], vf[DH / 16];
  load_row_frags<DH>(qkv + krow * a.ld_qkv + a.qkv_ko + hd * a.qkv_hs, kv, half, kf);
  load_row_frags<DH>(qkv + krow * a.ld_qkv + a.qkv_vo + hd * a.qkv_hs, kv, half, vf);

  f32x16 dk[DH / 32], dv[DH / 32];
#pragma unroll
  for (int i = 0; i < DH / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) dk[i][r] = dv[i][r] = 0.f;

  put_stats(qt0, lnext, dnext);
  for (int qt = qt0; qt < nqt; ++qt) {
    tiles_ready();
    if (qt + 1 < nqt) {
      load_stats(qt + 1, lnext, dnext);
      issue(qt + 1);
    }
    const bf16* sQ = sm + (qt & 1) * 2 * TILE;
    const bf16* sO = sQ + TILE;
    const float* pL = sL[qt & 1];
    const float* pD = sD[qt & 1];
    // one query block at a time (not unrolled), as in the dQ pass
#pragma unroll 1
    for (int qb = 0; qb < KR / 32; ++qb) {
      const int q0 = qt * KR + qb * 32;
      if (k0 >= S || q0 >= S) break;          // wave-uniform
      if (CAUSAL && q0 + 31 < k0) continue;
      // the read offsets are formed per block: kept across the loop they spill at d_head 128
      if constexpr (DH == 128) asm volatile("" : "+v"(rd.row), "+v"(rd.tr));
      const bool full = k0 + 32 <= S && q0 + 32 <= S && (!CAUSAL || k0 + 31 <= q0);
      f32x16 st, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) st[r] = dp[r] = 0.f;
#pragma unroll
      for (int s = 0; s < DH / 16; ++s) {
        st = mfma32(rd.frag(sQ, qb, s), kf[s], st);
        dp = mfma32(rd.frag(sO, qb, s), vf[s], dp);
      }
#pragma unroll
      for (int g = 0; g < 4; ++g) {  // queries q0 + 8g + 4*half + 0..3
        const float4 L = *reinterpret_cast<const float4*>(pL + qb * 32 + 8 * g + 4 * half);
        const float4 D = *reinterpret_cast<const float4*>(pD + qb * 32 + 8 * g + 4 * half);
        const float lv[4] = {L.x, L.y, L.z, L.w}, sv[4] = {D.x, D.y, D.z, D.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = 4 * g + e, qq = q0 + 8 * g + 4 * half + e;
          const bool ok = full || (kv && qq < S && (!CAUSAL || key <= qq));
          const float p = ok ? __builtin_amdgcn_exp2f(fmaf(st[r], sl2, -lv[e])) : 0.f;
          st[r] = p;
          dp[r] = p * (dp[r] - sv[e]);  // dS
        }
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 pf = pack8(st, j), sf = pack8(dp, j);
#pragma unroll
        for (int db = 0; db < DH / 32; ++db) {
          dv[db] = mfma32(rd.perm(sO, db, qb, j), pf, dv[db]);
          dk[db] = mfma32(rd.perm(sQ, db, qb, j), sf, dk[db]);
        }
      }
    }
    if (qt + 1 < nqt) put_stats(qt + 1, lnext, dnext);  // the other buffer: last read before this tile's barrier
  }
  tiles_ready();  // the tiles' space now takes the dK, then the dV rows
  if (k0 >= S) return;
  if (a.rope) unrotate<DH>(dk, min(key, S - 1), a.rope_tab, half);
  bf16* dst = static_cast<bf16*>(a.dqkv) + (long)(b * S + k0) * a.ld_dqkv + d + hd * DH;
  bf16* stage = sm + wave * 32 * (DH + 8);
  const bool nt = stream_out(3l * a.B * S * d * 2);
  store_rows_staged<DH>(dk, scale, half, lane, stage, dst, a.ld_dqkv, nt, S - k0);
  store_rows_staged<DH>(dv, 1.f, half, lane, stage, dst + d, a.ld_dqkv, nt, S - k0);
}

// Whole backward of one (batch, head) with S <= KT (one query block, one key
// tile), one workgroup: P and dS are formed once.  Wave w owns queries
// 32w..32w+31 (lane = query, as in the dQ pass): it computes its score and
// dP blocks against the K and V tiles, accumulates dQ and keeps P and dS
// packed in registers.  The K/V tile space is then reused for P (row-major
// [query][key]); each wave now owns keys 32w..32w+31 and reads its P^T
// fragments from that block with the LDS transpose read, for dV = P^T dO;
// then dS goes to the same space for dK = dS^T Q.  The LDS holds Q, dO and
// the K/V tiles (74 KB at d_head 64: two workgroups per CU).  The results leave
// through the dO tile as whole streamed rows: 384 of these at S 128, d_head 64
// took 20.3 us with 8-B pieces stored from the score layout, 17.2 us so.
template <int DH, bool CAUSAL, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(DH <= 64 ? 2 : 1))) void attn_bwd_fused_bf16(AttnArgs a) {
  static_assert(NW * 32 == KT, "one 32-row block per wave covers the tile");
  constexpr int TP = KT * (DH + 8), PP = KT + 8;
  static_assert(2 * TP >= KT * PP, "P fits in the K/V tile space");
  __shared__ __attribute__((aligned(16))) bf16 sQ[TP];
  __shared__ __attribute__((aligned(16))) bf16 sdO[TP];
  __shared__ __attribute__((aligned(16))) bf16 sKV[2 * TP];  // K, V; later P, then dS ([query][key], pitch PP)
  bf16* sK = sKV;
  bf16* sV = sKV + TP;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, half = lane >> 5, l32 = lane & 31;
  const int bh = xcd_block(blockIdx.y, gridDim.y), b = bh / a.H, hd = bh % a.H, S = a.S;
  const int d = a.H * DH;
  const float2* rtab = a.rope_tab;
  const float scale = rsqrtf((float)DH), sl2 = kLog2e * scale;
  const bf16* qkv = static_cast<const bf16*>(a.qkv);
  const bf16* dO = static_cast<const bf16*>(a.dout);

  // Q, dO, K, V tiles (rows >= S zero), this lane's O row
  // and its LSE, every global load issued before the first LDS store, none
  // conditional on a lane (rows past S read a valid row, masked afterwards).  The
  // prologue is bound by memory bandwidth (all workgroups load at once), so
  // dO is read once: the row sum D = rowsum(dO * O) takes it from the tile.
  const int q = wave * 32 + l32;
  const bool qv = q < S;
  const long qrow = (long)(b * S + (qv ? q : 0));
  TileLoad<DH, 64 * NW> tq, tdo, tk, tv;
  tq.issue(qkv, a.ld_qkv, hd * a.qkv_hs, b, S, 0);
  tdo.issue(dO, a.ld_do, hd * DH, b, S, 0);
  tk.issue(qkv, a.ld_qkv, a.qkv_ko + hd * a.qkv_hs, b, S, 0);
  tv.issue(qkv, a.ld_qkv, a.qkv_vo + hd * a.qkv_hs, b, S, 0);
  bf16x8 orw[DH / 16];
  {
    const bf16* orow = static_cast<const bf16*>(a.o) + qrow * a.ld_o + hd * DH;
#pragma unroll
    for (int s = 0; s < DH / 16; ++s) orw[s] = ld_frag(orow + 16 * s + 8 * half);  // qrow clamped
  }
  const float lse_raw = a.lse[(long)bh * S + (qv ? q : 0)];
  tq.store(sQ, S, 0);
  tdo.store(sdO, S, 0);
  tk.store(sK, S, 0);
  tv.store(sV, S, 0);
  __syncthreads();
  // the O row and the LSE were loaded last; masked only here, at their first use
  const float lse = qv ? lse_raw : 0.f;
  float dsum = 0.f;
#pragma unroll
  for (int s = 0; s < DH / 16; ++s) {
    float ov[8], dv[8];
    unpack_frag(orw[s], ov);
#pragma unroll
    for (int v = 0; v < 8; ++v) ov[v] = qv ? ov[v] : 0.f;
    unpack_frag(ld_frag(sdO + q * (DH + 8) + 16 * s + 8 * half), dv);  // rows >= S are zero
#pragma unroll
    for (int v = 0; v < 8; ++v) dsum += ov[v] * dv[v];
  }
  dsum += __shfl_xor(dsum, 32, 64);

  // ---- scores, P, dS and dQ (lane = query)
  const bool full = !CAUSAL && S == KT;
  bf16x8 pk[KT / 32][2], sk[KT / 32][2];
  f32x16 dq[DH / 32];
  {
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) dq[i][r] = 0.f;
#pragma unroll
    for (int kb = 0; kb < KT / 32; ++kb) {
      f32x16 st, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) st[r] = dp[r] = 0.f;
#pragma unroll
      for (int s = 0; s < DH / 16; ++s) {
        const bf16x8 qf = ld_frag(sQ + q * (DH + 8) + 16 * s + 8 * half);
        const bf16x8 df = ld_frag(sdO + q * (DH + 8) + 16 * s + 8 * half);
        st = mfma32(ld_frag(sK + (kb * 32 + l32) * (DH + 8) + 16 * s + 8 * half), qf, st);
        dp = mfma32(ld_frag(sV + (kb * 32 + l32) * (DH + 8) + 16 * s + 8 * half), df, dp);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = kb * 32 + perm_pos(r, half);
        const bool ok = full || (qv && key < S && (!CAUSAL || key <= q));
        const float p = ok ? __builtin_amdgcn_exp2f(fmaf(st[r], sl2, -lse)) : 0.f;
        st[r] = p;
        dp[r] = p * (dp[r] - dsum);  // dS
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        pk[kb][j] = pack8(st, j);
        sk[kb][j] = pack8(dp, j);
#pragma unroll
        for (int db = 0; db < DH / 32; ++db) dq[db] = mfma32(perm_frag<DH>(sK, db, kb, j, lane), sk[kb][j], dq[db]);
      }
    }
  }

  // a [query][key] block from the packed registers: register values 8j..8j+7
  // of key block kb are keys kb*32 + 16j + 4*half + {0..3, 8..11}
  auto put = [&](bf16x8 (&v)[KT / 32][2]) {
#pragma unroll
    for (int kb = 0; kb < KT / 32; ++kb)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const uint4 w = __builtin_bit_cast(uint4, v[kb][j]);
        bf16* row = sKV + q * PP + kb * 32 + 16 * j + 4 * half;
        *reinterpret_cast<uint2*>(row) = make_uint2(w.x, w.y);
        *reinterpret_cast<uint2*>(row + 8) = make_uint2(w.z, w.w);
      }
  };
  // dX[key][dim] += sum_q M[q][key] X[q][dim] over the whole tile (lane = key)
  auto tmul = [&](const bf16* sX, f32x16 (&acc)[DH / 32]) {
#pragma unroll
    for (int i = 0; i < DH / 32; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
#pragma unroll
    for (int qb = 0; qb < KT / 32; ++qb)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const bf16x8 mf = perm_frag<KT>(sKV, wave, qb, j, lane);
#pragma unroll
        for (int db = 0; db < DH / 32; ++db) acc[db] = mfma32(perm_frag<DH>(sX, db, qb, j, lane), mf, acc[db]);
      }
  };
  // The results leave as whole rows through the dO tile, each wave through its own
  // 32 rows, once every wave has read dO for the last time.  wave * 32 + lane % 32
  // is this lane's key as well as its query.
  bf16* stage = sdO + wave * 32 * (DH + 8);
  bf16* dst = static_cast<bf16*>(a.dqkv) + (long)(b * S + wave * 32) * a.ld_dqkv + hd * DH;
  const int n = S - wave * 32;
  const bool nt = stream_out(3l * a.B * S * d * 2);
  const int pos = min(q, S - 1);

  __syncthreads();  // every wave is done with K and V
  put(pk);
  __syncthreads();
  f32x16 dv[DH / 32];
  tmul(sdO, dv);
  __syncthreads();  // every wave is done with P and dO
  put(sk);
  if (a.rope) unrotate<DH>(dq, pos, rtab, half);
  store_rows_staged<DH>(dq, scale, half, lane, stage, dst, a.ld_dqkv, nt, n);
  store_rows_staged<DH>(dv, 1.f, half, lane, stage, dst + 2 * d, a.ld_dqkv, nt, n);
  __syncthreads();
  f32x16 dk[DH / 32];
  tmul(sQ, dk);
  if (a.rope) unrotate<DH>(dk, pos, rtab, half);
  store_rows_staged<DH>(dk, scale, half, lane, stage, dst + d, a.ld_dqkv, nt, n);
}

// ================================================================ fp32 (small stages)
// The fp32 stage is post-LN: bidirectional, no rotary embedding; head dim <= 128.
// Bound by latency (a few hundred tokens), so the work is cut into 16 own rows
// per workgroup (queries; keys in the dK/dV half of the backward), four per
// wave, against LDS tiles of 64 rows of the other side.  The dot products run
// with one tile row per lane, the sums over the tile with one head dim (or
// two) per lane, the probabilities passing through LDS between them.
// B 4, H 2, S 32, dh 64: forward 552 -> 8 us, backward 1413 -> 11 us
// (before: one thread per query, its row in scratch memory).
constexpr int F32_OWN = 16, F32_TILE = 64;

// rows r0 .. r0 + ROWS - 1 of one head into LDS (pitch DHM + 4), zero past
// row S and past column dh; every load of the tile in flight at once
template <int DHM, int ROWS>
struct RowsF32 {
  static constexpr int IT = ROWS * DHM / 256;
  float raw[IT];
  __device__ __forceinline__ void issue(const float* src, long ld, int S, int r0, int dh) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int idx = threadIdx.x + 256 * i, r = r0 + idx / DHM, c = idx % DHM;
      raw[i] = src[(long)min(r, S - 1) * ld + min(c, dh - 1)];
    }
  }
  __device__ __forceinline__ void store(float* dst, int S, int r0, int dh) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int idx = threadIdx.x + 256 * i, r = idx / DHM, c = idx % DHM;
      dst[r * (DHM + 4) + c] = r0 + r < S && c < dh ? raw[i] : 0.f;
    }
  }
};

// dot products of a wave's four own rows with this lane's tile row
template <int DHM>
__device__ __forceinline__ void dots_f32(const float* own, const float* tile, int lane, int dh, float s[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) s[i] = 0.f;
#pragma unroll 4
  for (int c = 0; c < dh; c += 4) {  // columns dh .. are zero
    const float4 t = *reinterpret_cast<const float4*>(tile + lane * (DHM + 4) + c);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 q = *reinterpret_cast<const float4*>(own + i * (DHM + 4) + c);
      s[i] = fmaf(q.x, t.x, s[i]);
      s[i] = fmaf(q.y, t.y, s[i]);
      s[i] = fmaf(q.z, t.z, s[i]);
      s[i] = fmaf(q.w, t.w, s[i]);
    }
  }
}

// acc[i][j] += sum over the tile rows r < n of p[i][r] tile[r][lane + 64 j]
// (p is zero from row n on)
template <int DHM>
__device__ __forceinline__ void sums_f32(const float (*p)[F32_TILE], const float* tile, int n, int lane,
                                         float (&acc)[4][DHM / 64]) {
#pragma unroll 4
  for (int r = 0; r < n; r += 4) {
    float4 w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) w[i] = *reinterpret_cast<const float4*>(&p[i][r]);
#pragma unroll
    for (int j = 0; j < DHM / 64; ++j) {
      float t[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) t[e] = tile[(r + e) * (DHM + 4) + lane + 64 * j];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        acc[i][j] = fmaf(w[i].x, t[0], acc[i][j]);
        acc[i][j] = fmaf(w[i].y, t[1], acc[i][j]);
        acc[i][j] = fmaf(w[i].z, t[2], acc[i][j]);
        acc[i][j] = fmaf(w[i].w, t[3], acc[i][j]);
      }
    }
  }
}

template <int DHM>
__global__ __launch_bounds__(256) void attn_fwd_f32(AttnArgs a) {
  constexpr int P = DHM + 4, ND = DHM / 64;
  __shared__ __attribute__((aligned(16))) float sQ[F32_OWN * P], sK[F32_TILE * P], sV[F32_TILE * P];
  __shared__ __attribute__((aligned(16))) float sP[F32_OWN][F32_TILE];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int S = a.S, dh = a.dh, nb = (S + F32_OWN - 1) / F32_OWN, bh = blockIdx.x / nb, b = bh / a.H, hd = bh % a.H;
  const int q0 = blockIdx.x % nb * F32_OWN;
  const float sl2 = kLog2e * rsqrtf((float)dh);
  const float* qkv = static_cast<const float*>(a.qkv) + (long)b * S * a.ld_qkv + hd * a.qkv_hs;
  RowsF32<DHM, F32_OWN> tq;
  RowsF32<DHM, F32_TILE> tk, tv;
  tq.issue(qkv, a.ld_qkv, S, q0, dh);
  tk.issue(qkv + a.qkv_ko, a.ld_qkv, S, 0, dh);
  tv.issue(qkv + a.qkv_vo, a.ld_qkv, S, 0, dh);
  tq.store(sQ, S, q0, dh);
  float m[4], l[4], o[4][ND];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    m[i] = -INFINITY;
    l[i] = 0.f;
#pragma unroll
    for (int j = 0; j < ND; ++j) o[i][j] = 0.f;
  }
  for (int k0 = 0; k0 < S; k0 += F32_TILE) {
    __syncthreads();
    tk.store(sK, S, k0, dh);
    tv.store(sV, S, k0, dh);
    __syncthreads();
    if (k0 + F32_TILE < S) {
      tk.issue(qkv + a.qkv_ko, a.ld_qkv, S, k0 + F32_TILE, dh);
      tv.issue(qkv + a.qkv_vo, a.ld_qkv, S, k0 + F32_TILE, dh);
    }
    float s[4];
    dots_f32<DHM>(sQ + wave * 4 * P, sK, lane, dh, s);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] = k0 + lane < S ? s[i] * sl2 : -INFINITY;
      const float mn = fmaxf(m[i], wave_max(s[i])), al = exp2f(m[i] - mn);
      s[i] = exp2f(s[i] - mn);
      l[i] = l[i] * al + wave_sum(s[i]);
      m[i] = mn;
#pragma unroll
      for (int j = 0; j < ND; ++j) o[i][j] *= al;
      sP[wave * 4 + i][lane] = s[i];  // read by this wave only
    }
    asm volatile("" ::: "memory");  // one wave's LDS operations run in order
    sums_f32<DHM>(sP + wave * 4, sV, min(F32_TILE, S - k0), lane, o);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int q = q0 + wave * 4 + i;
    if (q >= S) break;
    float* orow = static_cast<float*>(a.o) + (long)(b * S + q) * a.ld_o + hd * dh;
#pragma unroll
    for (int j = 0; j < ND; ++j)
      if (lane + 64 * j < dh) orow[lane + 64 * j] = o[i][j] / l[i];
    if (lane == 0) a.lse[(long)bh * S + q] = m[i] + log2f(l[i]);
  }
}

// Both halves of the backward in one launch (blockIdx.y): the dQ half owns
// queries (rows Q and dO) and walks the keys (K and V); the dK/dV half owns
// keys and walks the queries.  Each forms the row sums D = rowsum(dO * O) it
// needs itself.
template <int DHM>
__global__ __launch_bounds__(256) void attn_bwd_f32(AttnArgs a) {
  constexpr int P = DHM + 4, ND = DHM / 64;
  __shared__ __attribute__((aligned(16))) float sA[2][F32_OWN * P], sB[2][F32_TILE * P];
  __shared__ __attribute__((aligned(16))) float sS[F32_OWN][F32_TILE], sP[F32_OWN][F32_TILE];
  __shared__ float sL[F32_TILE], sD[F32_TILE];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int S = a.S, dh = a.dh, d = a.H * dh, nb = (S + F32_OWN - 1) / F32_OWN, bh = blockIdx.x / nb;
  const int b = bh / a.H, hd = bh % a.H, r0 = blockIdx.x % nb * F32_OWN;
  const bool keys = blockIdx.y != 0;
  const float scale = rsqrtf((float)dh), sl2 = kLog2e * scale;
  const float* q_ = static_cast<const float*>(a.qkv) + (long)b * S * a.ld_qkv + hd * a.qkv_hs;
  const float* do_ = static_cast<const float*>(a.dout) + (long)b * S * a.ld_do + hd * dh;
  const float* o_ = static_cast<const float*>(a.o) + (long)b * S * a.ld_o + hd * dh;
  const float* lse = a.lse + (long)bh * S;
  const float* own[2] = {keys ? q_ + a.qkv_ko : q_, keys ? q_ + a.qkv_vo : do_};
  const float* oth[2] = {keys ? q_ : q_ + a.qkv_ko, keys ? do_ : q_ + a.qkv_vo};
  const long ld_own2 = keys ? a.ld_qkv : a.ld_do, ld_oth2 = keys ? a.ld_do : a.ld_qkv;
  RowsF32<DHM, F32_OWN> ta0, ta1;
  RowsF32<DHM, F32_TILE> tb0, tb1;
  ta0.issue(own[0], a.ld_qkv, S, r0, dh);
  ta1.issue(own[1], ld_own2, S, r0, dh);
  tb0.issue(oth[0], a.ld_qkv, S, 0, dh);
  tb1.issue(oth[1], ld_oth2, S, 0, dh);
  ta0.store(sA[0], S, r0, dh);
  ta1.store(sA[1], S, r0, dh);
  __syncthreads();
  // own queries: D and the log-sum-exp of this wave's four rows
  float ol[4] = {0.f, 0.f, 0.f, 0.f}, od[4] = {0.f, 0.f, 0.f, 0.f};
  if (!keys) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = min(r0 + wave * 4 + i, S - 1);
      float s = 0.f;
#pragma unroll
      for (int j = 0; j < ND; ++j)
        if (lane + 64 * j < dh) s += sA[1][(wave * 4 + i) * P + lane + 64 * j] * o_[(long)r * a.ld_o + lane + 64 * j];
      od[i] = wave_sum(s);
      ol[i] = lse[r];
    }
  }
  float g1[4][ND], g2[4][ND];  // dQ; or dK and dV
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < ND; ++j) g1[i][j] = g2[i][j] = 0.f;
  for (int t0 = 0; t0 < S; t0 += F32_TILE) {
    __syncthreads();
    tb0.store(sB[0], S, t0, dh);
    tb1.store(sB[1], S, t0, dh);
    __syncthreads();
    if (t0 + F32_TILE < S) {
      tb0.issue(oth[0], a.ld_qkv, S, t0 + F32_TILE, dh);
      tb1.issue(oth[1], ld_oth2, S, t0 + F32_TILE, dh);
    }
    if (keys) {  // the tile's queries: four threads per row
      const int r = threadIdx.x / 4, row = min(t0 + r, S - 1);
      float s = 0.f;
#pragma unroll 8
      for (int c = threadIdx.x % 4; c < dh; c += 4) s += sB[1][r * P + c] * o_[(long)row * a.ld_o + c];
      s += __shfl_xor(s, 1, 64);
      s += __shfl_xor(s, 2, 64);
      if (threadIdx.x % 4 == 0) {
        sD[r] = s;
        sL[r] = lse[row];
      }
      __syncthreads();
    }
    float s[4], dp[4];
    dots_f32<DHM>(sA[0] + wave * 4 * P, sB[0], lane, dh, s);
    dots_f32<DHM>(sA[1] + wave * 4 * P, sB[1], lane, dh, dp);
    const bool ok = t0 + lane < S;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float p = ok ? exp2f(s[i] * sl2 - (keys ? sL[lane] : ol[i])) : 0.f;
      sS[wave * 4 + i][lane] = ok ? p * (dp[i] - (keys ? sD[lane] : od[i])) : 0.f;  // read by this wave only
      if (keys) sP[wave * 4 + i][lane] = p;
    }
    asm volatile("" ::: "memory");  // one wave's LDS operations run in order
    sums_f32<DHM>(sS + wave * 4, sB[0], min(F32_TILE, S - t0), lane, g1);
    if (keys) sums_f32<DHM>(sP + wave * 4, sB[1], min(F32_TILE, S - t0), lane, g2);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = r0 + wave * 4 + i;
    if (r >= S) break;
    float* dst = static_cast<float*>(a.dqkv) + (long)(b * S + r) * a.ld_dqkv + hd * dh;
#pragma unroll
    for (int j = 0; j < ND; ++j) {
      const int c = lane + 64 * j;
      if (c >= dh) continue;
      dst[(keys ? d : 0) + c] = g1[i][j] * scale;
      if (keys) dst[2 * d + c] = g2[i][j];
    }
  }
}

// ================================================================ launchers
static bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// four waves (128 queries or keys) per workgroup
constexpr int ATT_NW = 4;
constexpr int ATT_KR = 64;  // rows of the other side per tile

template <int DH>
static hipError_t fwd_dh(const AttnArgs& a, hipStream_t s) {
  dim3 grid((a.S + 32 * ATT_NW - 1) / (32 * ATT_NW), a.B * a.H), block(64 * ATT_NW);
  if (a.causal) RG_LAUNCH((attn_fwd_bf16<DH, true, ATT_NW, ATT_KR>), grid, block, 0, s, a);
  else RG_LAUNCH((attn_fwd_bf16<DH, false, ATT_NW, ATT_KR>), grid, block, 0, s, a);
  return hipGetLastError();
}
template <int DH>
static hipError_t bwd_dh(const AttnArgs& a, hipStream_t s) {
  dim3 grid((a.S + 32 * ATT_NW - 1) / (32 * ATT_NW), a.B * a.H), block(64 * ATT_NW);
  if (a.S <= KT) {  // one tile: the fused single-pass backward
    if (a.causal) RG_LAUNCH((attn_bwd_fused_bf16<DH, true, ATT_NW>), dim3(1, a.B * a.H), block, 0, s, a);
    else RG_LAUNCH((attn_bwd_fused_bf16<DH, false, ATT_NW>), dim3(1, a.B * a.H), block, 0, s, a);
    return hipGetLastError();
  }
  if (a.causal) {
    RG_LAUNCH((attn_bwd_dq_bf16<DH, true, ATT_NW, ATT_KR>), grid, block, 0, s, a);
    RG_LAUNCH((attn_bwd_dkdv_bf16<DH, true, ATT_NW, ATT_KR>), grid, block, 0, s, a);
  } else {
    RG_LAUNCH((attn_bwd_dq_bf16<DH, false, ATT_NW, ATT_KR>), grid, block, 0, s, a);
    RG_LAUNCH((attn_bwd_dkdv_bf16<DH, false, ATT_NW, ATT_KR>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

static hipError_t check(int dtype, const AttnArgs& a, bool bwd) {
  if (a.B <= 0 || a.S <= 0 || a.H <= 0 || !a.qkv || !a.o || !a.lse) return hipErrorInvalidValue;
  if (bwd && (!a.dout || !a.dsum || !a.dqkv)) return hipErrorInvalidValue;
  if (a.rope && (!a.rope_tab || a.rope_rows < a.S)) return hipErrorInvalidValue;
  if (a.rope && dtype != DT_BF16) return hipErrorInvalidValue;
  const int d = a.H * a.dh;
  const bool three_block = a.qkv_hs == a.dh && a.qkv_ko == d && a.qkv_vo == 2 * d;
  const bool per_head = a.qkv_hs == 3 * a.dh && a.qkv_ko == a.dh && a.qkv_vo == 2 * a.dh;
  if (!three_block && !(per_head && dtype == DT_BF16)) return hipErrorInvalidValue;
  if (dtype == DT_BF16) {
    if (a.dh != 64 && a.dh != 128) return hipErrorInvalidValue;
    if (a.ld_qkv % 8 || a.ld_o % 8 || !al16(a.qkv) || !al16(a.o)) return hipErrorInvalidValue;
    if (bwd && (a.ld_do % 8 || a.ld_dqkv % 8 || !al16(a.dout) || !al16(a.dqkv))) return hipErrorInvalidValue;
  } else {
    if (a.dh > 128 || a.dh % 2 || a.S > 4096 || a.causal || a.rope) return hipErrorInvalidValue;
  }
  return hipSuccess;
}

// the three-block Q | K | V order when no per-head layout is given
static AttnArgs with_layout(AttnArgs a) {
  if (a.qkv_hs == 0 && a.qkv_ko == 0 && a.qkv_vo == 0) {
    a.qkv_hs = a.dh;
    a.qkv_ko = a.H * a.dh;
    a.qkv_vo = 2 * a.H * a.dh;
  }
  return a;
}

hipError_t launch_attn_fwd(int dtype, const AttnArgs& a0, hipStream_t s) {
  const AttnArgs a = with_layout(a0);
  hipError_t e = check(dtype, a, false);
  if (e != hipSuccess) return e;
  if (dtype == DT_BF16) return a.dh == 64 ? fwd_dh<64>(a, s) : fwd_dh<128>(a, s);
  const dim3 grid((a.S + F32_OWN - 1) / F32_OWN * a.B * a.H), block(256);
  if (a.dh <= 64) RG_LAUNCH(attn_fwd_f32<64>, grid, block, 0, s, a);
  else RG_LAUNCH(attn_fwd_f32<128>, grid, block, 0, s, a);
  return hipGetLastError();
}

hipError_t launch_attn_bwd(int dtype, const AttnArgs& a0, hipStream_t s) {
  const AttnArgs a = with_layout(a0);
  hipError_t e = check(dtype, a, true);
  if (e != hipSuccess) return e;
  if (dtype == DT_BF16) return a.dh == 64 ? bwd_dh<64>(a, s) : bwd_dh<128>(a, s);
  const dim3 grid((a.S + F32_OWN - 1) / F32_OWN * a.B * a.H, 2), block(256);
  if (a.dh <= 64) RG_LAUNCH(attn_bwd_f32<64>, grid, block, 0, s, a);
  else RG_LAUNCH(attn_bwd_f32<128>, grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace rg
