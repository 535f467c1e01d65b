"""The GEMM launcher's own choice of a tile (csrc/gemm_tiles.h), compiled for the
host: the tiles that a bf16 stage's eight projection products take, and the
(call site, epilogue, tile) kernels that legal stages reach."""
import ctypes
import functools
import os
import subprocess
import tempfile

from paper_2502_19864_amd.build import CSRC

SITES = ("qkv_fwd", "o_fwd", "ffn_in_fwd", "ffn_out_fwd", "qkv_dx", "o_dx", "ffn_in_dx", "ffn_out_dx")
EPIS = {"bert": ("store", "store", "gelu", "store", "resid", "store", "resid", "dgelu"),
        "llama": ("rope", "store", "swiglu", "store", "store", "store", "store", "dswiglu")}
WIDTHS = (256, 512, 768, 1024, 2048, 3072, 4096)  # the d of a bf16 stage

SOURCE = r"""
#include "gemm_tiles.h"
using namespace rg;
static const Role SITE[8] = {R_QKV_FWD, R_O_FWD, R_FFN_IN_FWD, R_FFN_OUT_FWD, R_QKV_DX, R_O_DX, R_FFN_IN_DX, R_FFN_OUT_DX};
static const Epi EPI[2][8] = {
    {Epi::Store, Epi::Store, Epi::Gelu, Epi::Store, Epi::Resid, Epi::Store, Epi::Resid, Epi::DGelu},
    {Epi::Rope, Epi::Store, Epi::SwiGlu, Epi::Store, Epi::Store, Epi::Store, Epi::Store, Epi::DSwiGlu}};
extern "C" {
int n_cfgs() { return N_CFGS; }
void tile_of(int c, int* t) { t[0] = TILE[c].bm; t[1] = TILE[c].bn; t[2] = TILE[c].bk; t[3] = TILE[c].slots; }
int built(int llama, int site, int c) { return role_has(SITE[site], EPI[llama][site]) && cfg_has(SITE[site], EPI[llama][site], (Cfg)c); }
void choose(int llama, int T, int d, int F, int* cfg) {
  const int F2 = llama ? 2 * F : F;
  const int N[8] = {3 * d, d, F2, d, d, d, d, F}, K[8] = {d, d, d, F, 3 * d, d, F2, d};
  for (int i = 0; i < 8; ++i) cfg[i] = choose_tile(SITE[i], EPI[llama][i], T, N[i], K[i]);
}
// hit[site][tile] over FFN widths up to 16384 and token counts up to a stage's limit
void sweep(int llama, int d, unsigned char* hit) {
  int cfg[8];
  for (long F = 64; F <= 16384; F += F < 4096 ? 64 : 192)
    for (long T = 32; 3 * T * d <= 2000000000 && 2 * T * F <= 2000000000; T += T < 4096 ? 32 : T < 32768 ? 256 : 32768) {
      choose(llama, (int)T, d, (int)F, cfg);
      for (int i = 0; i < 8; ++i) hit[i * N_CFGS + cfg[i]] = 1;
    }
}
}
"""


@functools.lru_cache(None)
def lib():
    tmp = tempfile.mkdtemp(prefix="tile_choice_")
    src, so = os.path.join(tmp, "t.cpp"), os.path.join(tmp, "t.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I" + CSRC, src, "-o", so], check=True)
    return ctypes.CDLL(so)


@functools.lru_cache(None)
def names():
    """rows x columns; "/k64" the 64-wide k-tiles of a shape that has 128-wide ones
    too, "/2" the tiles that run two to a CU."""
    out = []
    for c in range(lib().n_cfgs()):
        t = (ctypes.c_int * 4)()
        lib().tile_of(c, t)
        bm, bn, bk, slots = t
        out.append(f"{bm}x{bn}" + ("/k64" if (bm, bn, bk) == (64, 128, 64) else "") + ("/2" if slots > 256 else ""))
    assert len(set(out)) == len(out)
    return tuple(out)


def kernels(arch, per_site):
    return {(s, e, names()[c]) for s, e, cs in zip(SITES, EPIS[arch], per_site) for c in cs}


def built(arch):
    """Every (call site, epilogue, tile) that is compiled."""
    ll = int(arch == "llama")
    return kernels(arch, [[c for c in range(lib().n_cfgs()) if lib().built(ll, i, c)] for i in range(8)])


def reached(arch):
    n = lib().n_cfgs()
    hit = (ctypes.c_ubyte * (8 * n))()
    for d in WIDTHS:
        lib().sweep(int(arch == "llama"), d, hit)
    return kernels(arch, [[c for c in range(n) if hit[i * n + c]] for i in range(8)])


def taken(arch, tokens, d, ffn, fused):
    """The kernels of one block's forward and full backward; fused: the QKV
    projection takes the attention into its epilogue, on a tile of its own."""
    cfg = (ctypes.c_int * 8)()
    lib().choose(int(arch == "llama"), tokens, d, ffn, cfg)
    return {k for k in kernels(arch, [[c] for c in cfg]) if not (fused and k[0] == "qkv_fwd")}
