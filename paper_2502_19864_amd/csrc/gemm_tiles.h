// The projection GEMMs' call sites, epilogues and bf16 tiles, and the choice among
// them.  Plain C++ without HIP: the choice can be compiled and swept on the host.
#pragma once

namespace rg {

enum class Epi {
  Store,    // out = acc (+ bias[n])
  Gelu,     // pre = acc (+ bias[n]); out2 = pre (if non-null); out = gelu(pre)
  Resid,    // out = acc + aux[m, n]
  DGelu,    // out = acc * gelu'(aux[m, n])
  SwiGlu,   // B rows packed [gate 32 | up 32] per 64; out[m, f] = silu(gate) * up,
            // out2[m, f] = gate, out2[m, half + f] = up (if non-null)
  DSwiGlu,  // acc = d(act)[m, f]; aux = [gate | up]; out[m, f] = d gate,
            // out[m, half + f] = d up
  Rope,     // bf16 QKV projection, no bias: out = acc with the rotary embedding
            // applied to columns < rope_cols (Q and K, heads of rope_dh
            // columns; row m is position m % rope_S)
  Attn,     // bf16 QKV projection with B rows in per-head order [Q_h K_h V_h]
            // (d_head 64) and M = sequences of 128 tokens: pre = acc + bias;
            // out = pre (if non-null); out2[:, 64h..64h+63] = softmax(Q_h K_h^T / 8) V_h
            // per sequence; lse[(seq * H + h) * 128 + query] (base 2, scaled scores)
};

// Names of the GEMM call sites (each gets its own kernel symbol).
enum Role {
  R_QKV_FWD, R_O_FWD, R_FFN_IN_FWD, R_FFN_OUT_FWD,
  R_QKV_DX, R_O_DX, R_FFN_IN_DX, R_FFN_OUT_DX, N_ROLES
};

// epilogues each call site uses (only these are instantiated)
constexpr bool role_has(Role r, Epi e) {
  switch (r) {
    case R_QKV_FWD: return e == Epi::Store || e == Epi::Attn || e == Epi::Rope;
    case R_O_FWD: case R_FFN_OUT_FWD: case R_O_DX: return e == Epi::Store;
    case R_FFN_IN_FWD: return e == Epi::Gelu || e == Epi::SwiGlu;
    case R_QKV_DX: case R_FFN_IN_DX: return e == Epi::Resid || e == Epi::Store;
    case R_FFN_OUT_DX: return e == Epi::DGelu || e == Epi::DSwiGlu;
    default: return false;
  }
}

// Tile shapes of the pipelined kernel.  A launch takes as long as its rounds of
// workgroups, and a round costs about f + r K / 64 us (f: launch, first loads,
// epilogue), so the tile with the least sum over its rounds is taken.  The
// figures are fitted to launches whose operands come from memory, as they do
// inside a stage; each shape wins somewhere, in us (against the next best here):
//   256x256  4096 x 4096 x 1024   34.6 (256x128 39.8)
//   256x192  4096 x 3072 x 1024   28.8 (128x192 29.1)
//   256x128  2048 x 4096 x 11008   155 (128x128 205)
//   128x192  4096 x 3072 x 768    22.2 (256x192 23.7); four stages for one
//            tile per CU: 1827 x 3072 x 768 13.5 (256x128 14.7)
//   128x128  4096 x 1024 x 4096   39.0 (128x192 45.1); two stages for two per CU:
//            4096 x 5120 x 256, where 256-row tiles leave their last round short
//   128x96   4096 x 768 x 3072    27.6 (128x128 31.6)
//   64x128   1827 x 768 x 3072    20.8 (128x96 26.2)
//   64x64    256 x 4096 x 4096    20.4 (64x128 27.2)
//   32x64    100 x 4096 x 11008   34.4 (32x32 38.6, 64x64 46.2)
//   32x32    37 x 768 x 3072       8.0 (32x64 10.3, 64x64 13.7)
// The last two are one wave wide and deal K to four wave groups (KG): the whole
// tile from fragments read once, and four waves' loads in flight.  On larger
// tiles KG brought nothing (128x96 27.6 -> 28.6).
// slots: workgroups the chip holds.  Where that is 512 (two per CU), (f, r) are those of
// a full round and (f1, r1) those of one with at most a workgroup per CU.
enum Cfg {
  C_32x32, C_32x64, C_64x64, C_64x128, C_64x128_K64, C_128x96, C_128x128, C_128x128_2, C_128x192, C_128x192_2,
  C_256x128, C_256x192, C_256x256, N_CFGS
};
struct Tile { int bm, bn, bk, slots; float f, r, f1, r1; };
constexpr Tile TILE[N_CFGS] = {
    {32, 32, 128, 512, 2.8f, .21f, 2.8f, .11f}, {32, 64, 128, 256, 1.8f, .19f, 0, 0},
    {64, 64, 128, 256, 2.5f, .27f, 0, 0},
    {64, 128, 128, 256, 2.2f, .40f, 0, 0},     {64, 128, 64, 256, 2.3f, .43f, 0, 0},
    {128, 96, 64, 256, 3.9f, .49f, 0, 0},      {128, 128, 64, 256, 3.3f, .56f, 0, 0},
    {128, 128, 64, 512, 4.5f, .96f, 3.0f, .8f}, {128, 192, 64, 256, 4.6f, .73f, 0, 0},
    {128, 192, 64, 512, 4.6f, 1.47f, 3.9f, .97f}, {256, 128, 64, 256, 3.5f, .89f, 0, 0},
    {256, 192, 64, 256, 8.5f, 1.27f, 0, 0},    {256, 256, 64, 256, 9.0f, 1.6f, 0, 0}};

// Tiles a call site can take.  SwiGLU needs gate/up block pairs (64 columns) in a
// wave, the rotary epilogue whole heads (128 columns) in a tile.  The 64-wide k-tiles
// of 64x128 serve a K that 128 does not divide, which only the post-LN or plain
// products over the FFN width have (every other K is d, 3 d or 2 F).  dSwiGLU's
// epilogue term below leaves it no shape where 256x128 or 256x192 is the least.
constexpr bool cfg_has(Role R, Epi E, Cfg c) {
  switch (c) {
    case C_64x128_K64: return (R == R_FFN_OUT_FWD && E == Epi::Store) || (R == R_FFN_IN_DX && E == Epi::Resid);
    case C_256x128: return E != Epi::DSwiGlu;
    case C_256x192: return E != Epi::DSwiGlu && E != Epi::SwiGlu && E != Epi::Rope;
    case C_64x128: case C_128x128: case C_128x128_2: case C_256x256: return true;
    default: return E != Epi::SwiGlu && E != Epi::Rope;
  }
}

// the tile of C[M, N] = A[M, K] B[N, K]^T at call site R; K a multiple of 64
inline Cfg choose_tile(Role R, Epi E, int M, int N, int K) {
  Cfg best = C_128x128;
  double least = 1e30;
  for (int c = 0; c < N_CFGS; ++c) {
    const Tile& t = TILE[c];
    if (!cfg_has(R, E, (Cfg)c) || K % t.bk) continue;
    const long n = (long)((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn), full = n / t.slots, rem = n % t.slots;
    // dSwiGLU moves 6 B more per output than the others, which a tile alone on its CU does
    // not hide (about 20 GB/s a CU): 2048 x 11008 x 4096 on 256x192 was 17 us slower than
    // on 128x192, two per CU
    const double epi = E == Epi::DSwiGlu && t.slots == 256 ? t.bm * t.bn * 6 / 20e3 : 0.;
    const double k = K / 64, round = t.f + epi + t.r * k;
    const double us = full * round + (rem == 0 ? 0. : (t.slots > 256 && rem <= 256) ? t.f1 + t.r1 * k : round);
    if (us < least) { least = us; best = (Cfg)c; }
  }
  return best;
}

}  // namespace rg
