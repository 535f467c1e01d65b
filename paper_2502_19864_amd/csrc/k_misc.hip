// Row-wise norms (RMSNorm, and the vectorised LayerNorm / RMSNorm rows of the
// wide adapters), parameter layout kernels, the adapter update and the
// initiator's loss helpers.
#include <algorithm>
#include <initializer_list>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace rg {

template <typename T>
__device__ float blk_sum(float v, float* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float t = 0.f;
  for (int w = 0; w < nw; ++w) t += red[w];
  return t;
}

// ---------------------------------------------------------------- row norms, bf16, vectorised
// One 256-thread workgroup per row, eight features per 16-B access (d <= 4096,
// so at most two per thread).
constexpr int NORM_NPT = 2;
__device__ __forceinline__ float block_sum256(float v, float* red) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  const float t = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return t;
}
__device__ __forceinline__ void ld8f(const bf16* p, float v[8]) { unpack_frag(ld_frag(p), v); }
__device__ __forceinline__ void st8f(bf16* p, const float v[8], bool nt) { st16(p, pack_frag(v), nt); }

// h = x1 (+ x2); LN: out = LN(h) g + b (out may alias x1); RMS: out = h (when
// x2 is given) and out_norm = RMSNorm(h) g; None: out = h.  xhat, rstd stashed
// when given.
__global__ __launch_bounds__(256) void norm_rows_fwd_bf16(int d, float eps, Norm norm, const bf16* x1,
                                                             const bf16* x2, const bf16* gamma, const bf16* beta,
                                                             bf16* out, bf16* out_norm, bf16* xhat, float* rstd) {
  __shared__ float red[4];
  const long row = (long)blockIdx.x * d;
  const int nc = d / 8;
  const bool nt = stream_out((long)gridDim.x * d * 2);  // one row per workgroup
  // every load up front, none conditional on a lane or an operand: a chunk past the row
  // reads chunk 0, an absent operand reads x1 (gamma) instead, masked afterwards; so no
  // load waits for the one before it
  const bf16* x2p = x2 ? x2 : x1;
  const bf16* gp = gamma ? gamma : x1;
  const bf16* bp = (norm == Norm::LN && beta) ? beta : gp;
  bf16x8 r1[NORM_NPT], r2[NORM_NPT], rg[NORM_NPT], rb[NORM_NPT];
#pragma unroll
  for (int i = 0; i < NORM_NPT; ++i) {
    const int c = threadIdx.x + 256 * i, cc = c < nc ? c : 0;
    r1[i] = ld_frag(x1 + row + 8 * cc);
    r2[i] = ld_frag(x2p + row + 8 * cc);
    rg[i] = ld_frag(gp + 8 * cc);
    rb[i] = ld_frag(bp + 8 * cc);
  }
  float v[NORM_NPT][8];
#pragma unroll
  for (int i = 0; i < NORM_NPT; ++i) {
    float y[8];
    unpack_frag(r1[i], v[i]);
    unpack_frag(r2[i], y);
    if (x2)
#pragma unroll
      for (int q = 0; q < 8; ++q) v[i][q] += y[q];
  }
  if (norm == Norm::None || (norm == Norm::RMS && x2)) {
#pragma unroll
    for (int i = 0; i < NORM_NPT; ++i) {
      const int c = threadIdx.x + 256 * i;
      if (c < nc) st8f(out + row + 8 * c, v[i], nt);
    }
    if (norm == Norm::None) return;
  }
  float mean = 0.f;
  if (norm == Norm::LN) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NORM_NPT; ++i)
      if (threadIdx.x + 256 * i < nc)
#pragma unroll
        for (int q = 0; q < 8; ++q) s += v[i][q];
    mean = block_sum256(s, red) / (float)d;
  }
  float s2 = 0.f;
#pragma unroll
  for (int i = 0; i < NORM_NPT; ++i)
    if (threadIdx.x + 256 * i < nc)
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const float c = v[i][q] - mean;
        s2 += c * c;
      }
  const float rs = rsqrtf(block_sum256(s2, red) / (float)d + eps);
  if (rstd && threadIdx.x == 0) rstd[blockIdx.x] = rs;
  bf16* dst = norm == Norm::LN ? out : out_norm;
#pragma unroll
  for (int i = 0; i < NORM_NPT; ++i) {
    const int c = threadIdx.x + 256 * i;
    if (c >= nc) continue;
    float xh[8], g[8], b[8], o[8];
    unpack_frag(rg[i], g);
    unpack_frag(rb[i], b);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      xh[q] = (v[i][q] - mean) * rs;
      o[q] = xh[q] * g[q] + (norm == Norm::LN ? b[q] : 0.f);
    }
    st8f(dst + row + 8 * c, o, nt);
    if (xhat) st8f(xhat + row + 8 * c, xh, nt);
  }
}

// dz = [dres +] rstd (g*gin - [mean(g*gin)] - xhat mean(g*gin*xhat)), LN or RMS
__global__ __launch_bounds__(256) void norm_rows_bwd_bf16(int d, Norm norm, const bf16* gin, const bf16* xhat,
                                                             const float* rstd, const bf16* gamma,
                                                             const bf16* dres, bf16* dz) {
  __shared__ float red[4];
  const long row = (long)blockIdx.x * d;
  const int nc = d / 8;
  const bool nt = stream_out((long)gridDim.x * d * 2);
  float gg[NORM_NPT][8], xh[NORM_NPT][8];
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int i = 0; i < NORM_NPT; ++i) {
    const int c = threadIdx.x + 256 * i;
    if (c >= nc) continue;
    float g[8];
    ld8f(gin + row + 8 * c, gg[i]);
    ld8f(xhat + row + 8 * c, xh[i]);
    ld8f(gamma + 8 * c, g);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      gg[i][q] *= g[q];
      s1 += gg[i][q];
      s2 += gg[i][q] * xh[i][q];
    }
  }
  const float m1 = norm == Norm::LN ? block_sum256(s1, red) / (float)d : 0.f;
  const float m2 = block_sum256(s2, red) / (float)d, rs = rstd[blockIdx.x];
#pragma unroll
  for (int i = 0; i < NORM_NPT; ++i) {
    const int c = threadIdx.x + 256 * i;
    if (c >= nc) continue;
    float r[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, o[8];
    if (norm == Norm::RMS) ld8f(dres + row + 8 * c, r);
#pragma unroll
    for (int q = 0; q < 8; ++q) o[q] = r[q] + rs * (gg[i][q] - m1 - xh[i][q] * m2);
    st8f(dz + row + 8 * c, o, nt);
  }
}

static bool al16p(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

hipError_t launch_norm_rows_fwd(int T, int d, float eps, Norm norm, const void* x1, const void* x2, const void* gamma,
                                const void* beta, void* out, void* out_norm, void* xhat, float* rstd, hipStream_t s) {
  if (T < 0 || d <= 0 || d % 8 || d > 256 * 8 * NORM_NPT || !x1) return hipErrorInvalidValue;
  if (norm != Norm::None && !gamma) return hipErrorInvalidValue;
  if (norm == Norm::LN && (!beta || !out)) return hipErrorInvalidValue;
  if (norm == Norm::RMS && !out_norm) return hipErrorInvalidValue;
  if ((norm == Norm::None || (norm == Norm::RMS && x2)) && !out) return hipErrorInvalidValue;
  for (const void* p : {x1, x2, gamma, beta, static_cast<const void*>(out), static_cast<const void*>(out_norm),
                        static_cast<const void*>(xhat)})
    if (p && !al16p(p)) return hipErrorInvalidValue;
  if (T == 0) return hipSuccess;
  RG_LAUNCH(norm_rows_fwd_bf16, dim3(T), dim3(256), 0, s, d, eps, norm, static_cast<const bf16*>(x1),
            static_cast<const bf16*>(x2), static_cast<const bf16*>(gamma), static_cast<const bf16*>(beta),
            static_cast<bf16*>(out), static_cast<bf16*>(out_norm), static_cast<bf16*>(xhat), rstd);
  return hipGetLastError();
}

hipError_t launch_norm_rows_bwd(int T, int d, Norm norm, const void* gin, const void* xhat, const float* rstd,
                                const void* gamma, const void* dres, void* dz, hipStream_t s) {
  if (T < 0 || d <= 0 || d % 8 || d > 256 * 8 * NORM_NPT || norm == Norm::None) return hipErrorInvalidValue;
  if (!gin || !xhat || !rstd || !gamma || !dz || (norm == Norm::RMS && !dres)) return hipErrorInvalidValue;
  for (const void* p : {gin, xhat, gamma, dres, static_cast<const void*>(dz)})
    if (p && !al16p(p)) return hipErrorInvalidValue;
  if (T == 0) return hipSuccess;
  RG_LAUNCH(norm_rows_bwd_bf16, dim3(T), dim3(256), 0, s, d, norm, static_cast<const bf16*>(gin),
            static_cast<const bf16*>(xhat), rstd, static_cast<const bf16*>(gamma), static_cast<const bf16*>(dres),
            static_cast<bf16*>(dz));
  return hipGetLastError();
}

hipError_t launch_rms_fwd(int dtype, int T, int d, float eps, const void* x, const void* g, void* out,
                          void* xhat, float* rstd, hipStream_t s) {
  // bf16 only (the pre-RMS block has no fp32 stage); every bf16 width (d a
  // multiple of 256 up to 4096) and the stage's 16-B aligned buffers take the
  // vectorised row kernel
  if (T < 0 || d <= 0 || !x || !g || !out) return hipErrorInvalidValue;
  if (dtype != DT_BF16 || d % 8 || d > 256 * 8 * NORM_NPT || !al16p(x) || !al16p(g) || !al16p(out) ||
      (xhat && !al16p(xhat)))
    return hipErrorInvalidValue;
  if (T == 0) return hipSuccess;
  return launch_norm_rows_fwd(T, d, eps, Norm::RMS, x, nullptr, g, nullptr, nullptr, out, xhat, rstd, s);
}

hipError_t launch_rms_bwd(int dtype, int T, int d, const void* dn, const void* dres, const void* xhat,
                          const float* rstd, const void* g, void* dx, hipStream_t s) {
  // bf16 only, as the forward
  if (T < 0 || d <= 0 || !dn || !dres || !xhat || !rstd || !g || !dx) return hipErrorInvalidValue;
  if (dtype != DT_BF16 || d % 8 || d > 256 * 8 * NORM_NPT || !al16p(dn) || !al16p(dres) || !al16p(xhat) ||
      !al16p(g) || !al16p(dx))
    return hipErrorInvalidValue;
  if (T == 0) return hipSuccess;
  return launch_norm_rows_bwd(T, d, Norm::RMS, dn, xhat, rstd, g, dres, dx, s);
}

// ---------------------------------------------------------------- layouts
// out[c', r] = in[r, c] with c' = c, or, with perm_dh > 0, the per-head order
// of a [Q | K | V] column block: column p * (cols / 3) + h * perm_dh + i goes
// to row (3 h + p) * perm_dh + i.
__device__ __forceinline__ int perm_col(int c, int cols, int perm_dh) {
  if (perm_dh <= 0) return c;
  const int blk = cols / 3, p = c / blk, rem = c % blk, h = rem / perm_dh, i = rem % perm_dh;
  return (3 * h + p) * perm_dh + i;
}

template <typename Ti, typename To>
__global__ __launch_bounds__(256) void transpose_k(const Ti* in, int rows, int cols, To* out, int perm_dh) {
  __shared__ float tile[32][33];
  const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32, tx = threadIdx.x % 32, ty = threadIdx.x / 32;
  for (int i = ty; i < 32; i += 8) {
    const int r = r0 + i, c = c0 + tx;
    tile[i][tx] = (r < rows && c < cols) ? St<Ti>::ld(in, (long)r * cols + c) : 0.f;
  }
  __syncthreads();
  for (int i = ty; i < 32; i += 8) {
    const int c = c0 + i, r = r0 + tx;
    if (c < cols && r < rows) St<To>::st(out, (long)perm_col(c, cols, perm_dh) * rows + r, tile[tx][i]);
  }
}

hipError_t launch_transpose(int in_dtype, int out_dtype, const void* in, int rows, int cols, void* out,
                            hipStream_t s, int perm_dh) {
  if (!in || !out || rows <= 0 || cols <= 0) return hipErrorInvalidValue;
  if (perm_dh > 0 && (cols % 3 || (cols / 3) % perm_dh)) return hipErrorInvalidValue;
  const dim3 grid((cols + 31) / 32, (rows + 31) / 32), block(256);
  if (in_dtype == DT_F32 && out_dtype == DT_F32)
    RG_LAUNCH((transpose_k<float, float>), grid, block, 0, s, (const float*)in, rows, cols, (float*)out, perm_dh);
  else if (in_dtype == DT_BF16 && out_dtype == DT_BF16)
    RG_LAUNCH((transpose_k<bf16, bf16>), grid, block, 0, s, (const bf16*)in, rows, cols, (bf16*)out, perm_dh);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <typename T>
__global__ __launch_bounds__(256) void pack_swiglu_k(const T* wgu, int d, int F, T* out) {
  const long n = 2L * F * d;
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (long)gridDim.x * blockDim.x) {
    const int p = (int)(idx / d), i = (int)(idx % d);
    const int blk = p / 64, w = p % 64;
    const int col = w < 32 ? blk * 32 + w : F + blk * 32 + (w - 32);
    out[idx] = wgu[(long)i * 2 * F + col];
  }
}

hipError_t launch_pack_swiglu(int dtype, const void* w_gu, int d, int F, void* out, hipStream_t s) {
  if (!w_gu || !out || d <= 0 || F <= 0 || F % 32) return hipErrorInvalidValue;
  const dim3 grid(4096), block(256);
  if (dtype != DT_BF16) return hipErrorInvalidValue;  // the SwiGLU block has no fp32 stage
  RG_LAUNCH(pack_swiglu_k<bf16>, grid, block, 0, s, (const bf16*)w_gu, d, F, (bf16*)out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- adapter update
// Element idx < d*m is W_down[i][j] (i = idx / m, j = idx % m); the rest is
// W_up[j][i].  Writes the working copies W, W^T in the stage dtype.  The
// slots of one launch travel by value (blockIdx.y selects one).
template <typename T, bool UPDATE>
__global__ __launch_bounds__(256) void adapter_update_k(AdapterSlotBatch batch, int d, int m, float lr) {
  const AdapterSlot& sl = batch.s[blockIdx.y];
  if (!sl.w_down) return;  // a block without this adapter (single placement)
  const long n = (long)d * m;
  for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < 2 * n; idx += (long)gridDim.x * blockDim.x) {
    if (idx < n) {
      const int i = (int)(idx / m), j = (int)(idx % m);
      float w = sl.w_down[idx];
      if (UPDATE) {
        w -= lr * sl.g_down[idx];
        sl.w_down[idx] = w;
        sl.g_down[idx] = 0.f;
      }
      if constexpr (std::is_same_v<T, float>) {
        St<T>::st(static_cast<T*>(sl.wdn), idx, w);
        St<T>::st(static_cast<T*>(sl.wdn_t), (long)j * d + i, w);
      } else {  // fragment-packed: W_down in layout B, W_down^T in layout A
        St<T>::st(static_cast<T*>(sl.wdn), pack_b_idx(i, j, d), w);
        St<T>::st(static_cast<T*>(sl.wdn_t), pack_a_idx(j, i, d), w);
      }
    } else {
      const long k = idx - n;
      const int j = (int)(k / d), i = (int)(k % d);
      float w = sl.w_up[k];
      if (UPDATE) {
        w -= lr * sl.g_up[k];
        sl.w_up[k] = w;
        sl.g_up[k] = 0.f;
      }
      if constexpr (std::is_same_v<T, float>) {
        St<T>::st(static_cast<T*>(sl.wup), k, w);
        St<T>::st(static_cast<T*>(sl.wup_t), (long)i * m + j, w);
      } else {  // W_up in layout A, W_up^T in layout B
        St<T>::st(static_cast<T*>(sl.wup), pack_a_idx(j, i, d), w);
        St<T>::st(static_cast<T*>(sl.wup_t), pack_b_idx(i, j, d), w);
      }
    }
  }
}

template <bool UPDATE>
static hipError_t adapter_update(int dtype, const AdapterSlot* slots, int n_slots, int d, int m, float lr,
                                 hipStream_t s) {
  if ((!slots && n_slots) || n_slots < 0 || d <= 0 || m <= 0) return hipErrorInvalidValue;
  const long n = 2L * d * m;
  const unsigned gx = (unsigned)((n + 255) / 256 < 256 ? (n + 255) / 256 : 256);
  for (int i0 = 0; i0 < n_slots; i0 += ADAPTER_SLOT_BATCH) {
    AdapterSlotBatch b{};
    const int k = n_slots - i0 < ADAPTER_SLOT_BATCH ? n_slots - i0 : ADAPTER_SLOT_BATCH;
    for (int i = 0; i < k; ++i) b.s[i] = slots[i0 + i];
    const dim3 grid(gx, k), block(256);
    if (dtype == DT_BF16) RG_LAUNCH((adapter_update_k<bf16, UPDATE>), grid, block, 0, s, b, d, m, lr);
    else RG_LAUNCH((adapter_update_k<float, UPDATE>), grid, block, 0, s, b, d, m, lr);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_adapter_sgd(int dtype, const AdapterSlot* slots, int n_slots, int d, int m, float lr,
                              hipStream_t s) {
  return adapter_update<true>(dtype, slots, n_slots, d, m, lr, s);
}
hipError_t launch_adapter_sync(int dtype, const AdapterSlot* slots, int n_slots, int d, int m,
                               hipStream_t s) {
  return adapter_update<false>(dtype, slots, n_slots, d, m, 0.f, s);
}

// ---------------------------------------------------------------- losses
// Mean squared error: bound by memory (three passes of n elements).  Up to
// MSE_ONE_BYTES per tensor one workgroup does it all.  Larger tensors take
// many workgroups and, with no workspace in the call, keep their partial sums
// in the first floats of dY itself: mse_k writes every other element of dY,
// then mse_finish_k adds the partials (a fixed order: the same bits every call)
// and writes the elements they stood in.  Eight (four) elements per 16-B access
// when the pointers allow it, U accesses in flight.
// 3.1 M bf16 elements (32 x 128 x 768): 1007 -> 5.7 us (18.9 MB, 3.3 TB/s).  One
// workgroup against many, per call, at 64, 128 and 224 KB per tensor: replayed from
// a graph 4.3 and 4.9, 5.9 and 4.9, 8.7 and 4.9 us; waited for 17.9 and 19.5, 19.6
// and 19.5, 22.3 and 19.5; in a loop that the host holds up, where the second
// launch counts, 6.4 and 10.3, 6.4 and 10.4, 8.4 and 10.5.  The line lies where a
// call that is waited for takes the same.
constexpr long MSE_ONE_BYTES = 128 << 10;
constexpr int MSE_MAX_WG = 1024;  // partial sums: one per thread of mse_finish_k
template <typename T, int NT, int U>
__global__ __launch_bounds__(NT) void mse_k(const T* y, const T* t, long n, T* dy, float* out, long skip, bool vec) {
  __shared__ float red[NT / 64];
  constexpr int VE = 16 / sizeof(T);
  const bool nt = stream_out(n * (long)sizeof(T));  // dY streamed (common.h)
  const long stride = (long)gridDim.x * NT, nvec = vec ? n / VE : 0;
  const float sc = 2.f / (float)n;
  float s = 0.f;
  for (long v0 = (long)blockIdx.x * NT + threadIdx.x; v0 < nvec; v0 += U * stride) {
    uint4 a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {  // past the end: the first vector again, masked below
      const long v = v0 + u * stride < nvec ? v0 + u * stride : v0;
      a[u] = reinterpret_cast<const uint4*>(y)[v];
      b[u] = reinterpret_cast<const uint4*>(t)[v];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long v = v0 + u * stride;
      if (v >= nvec) break;
      T o[VE];
#pragma unroll
      for (int e = 0; e < VE; ++e) {
        const float diff = St<T>::ld(reinterpret_cast<const T*>(&a[u]), e) - St<T>::ld(reinterpret_cast<const T*>(&b[u]), e);
        St<T>::st(o, e, sc * diff);
        s += diff * diff;
      }
      uint4 q;
      __builtin_memcpy(&q, o, 16);
      if (v * VE >= skip) st16(reinterpret_cast<uint4*>(dy) + v, __builtin_bit_cast(bf16x8, q), nt);
    }
  }
  for (long i = nvec * VE + (long)blockIdx.x * NT + threadIdx.x; i < n; i += stride) {
    const float diff = St<T>::ld(y, i) - St<T>::ld(t, i);
    if (i >= skip) St<T>::st(dy, i, sc * diff);
    s += diff * diff;
  }
  s = blk_sum<T>(s, red);
  // one workgroup: the loss itself; else this workgroup's partial sum
  if (out && threadIdx.x == 0) out[blockIdx.x] = gridDim.x == 1 ? s / (float)n : s;
}

template <typename T>
__global__ __launch_bounds__(MSE_MAX_WG) void mse_finish_k(const T* y, const T* t, long n, T* dy, const float* part,
                                                           int nwg, float* loss, long skip) {
  __shared__ float red[MSE_MAX_WG / 64];
  const float s = blk_sum<T>((int)threadIdx.x < nwg ? part[threadIdx.x] : 0.f, red);
  if (threadIdx.x == 0) *loss = s / (float)n;
  // every partial has been read (the sum's barriers): dY's own values now
  const float sc = 2.f / (float)n;
  for (long i = threadIdx.x; i < skip; i += MSE_MAX_WG) St<T>::st(dy, i, sc * (St<T>::ld(y, i) - St<T>::ld(t, i)));
}

// dY may be clear of an input or in its place, element on element; shifted over it,
// threads would overwrite elements that others have yet to read
bool mse_dy_ok(const void* y, const void* t, const void* dy, size_t bytes) {
  const uintptr_t pd = reinterpret_cast<uintptr_t>(dy);
  for (const void* in : {y, t}) {
    const uintptr_t p = reinterpret_cast<uintptr_t>(in);
    if (p != pd && p < pd + bytes && pd < p + bytes) return false;
  }
  return true;
}

template <typename T>
static hipError_t mse(const T* y, const T* t, long n, T* dy, float* loss, hipStream_t s) {
  const uintptr_t py = reinterpret_cast<uintptr_t>(y), pt = reinterpret_cast<uintptr_t>(t),
                  pd = reinterpret_cast<uintptr_t>(dy), bytes = (uintptr_t)n * sizeof(T);
  const bool vec = ((py | pt | pd) & 15u) == 0;
  const bool inplace = pd == py || pd == pt;  // the partial sums would overwrite inputs
  constexpr int NT = 256, U = 2;
  constexpr long VE = 16 / sizeof(T);
  if ((long)bytes <= MSE_ONE_BYTES || inplace) {
    RG_LAUNCH((mse_k<T, 1024, 4>), dim3(1), dim3(1024), 0, s, y, t, n, dy, loss, 0L, vec);
    return hipGetLastError();
  }
  const long want = (n / VE + NT * U - 1) / (NT * U);
  const int nwg = (int)(want < MSE_MAX_WG ? want : MSE_MAX_WG);
  float* part = reinterpret_cast<float*>((pd + 3) & ~(uintptr_t)3);
  // elements the partials cover, in whole vectors (MSE_ONE_BYTES keeps that far below n)
  const long skip = loss ? ((long)((reinterpret_cast<uintptr_t>(part + nwg) - pd + sizeof(T) - 1) / sizeof(T)) + VE - 1) / VE * VE : 0;
  RG_LAUNCH((mse_k<T, NT, U>), dim3(nwg), dim3(NT), 0, s, y, t, n, dy, loss ? part : nullptr, skip, vec);
  if (loss) RG_LAUNCH(mse_finish_k<T>, dim3(1), dim3(MSE_MAX_WG), 0, s, y, t, n, dy, part, nwg, loss, skip);
  return hipGetLastError();
}

hipError_t launch_mse(int dtype, const void* y, const void* t, long n, void* dy, float* loss, hipStream_t s) {
  if (!y || !t || !dy || n <= 0 || !mse_dy_ok(y, t, dy, n * (dtype == DT_BF16 ? 2 : 4))) return hipErrorInvalidValue;
  if (dtype == DT_BF16) return mse(static_cast<const bf16*>(y), static_cast<const bf16*>(t), n, static_cast<bf16*>(dy), loss, s);
  return mse(static_cast<const float*>(y), static_cast<const float*>(t), n, static_cast<float*>(dy), loss, s);
}

// Initiator head (Alg. 1: the initiator computes the loss and updates the
// head): a linear layer on position 0 of each sequence, softmax
// cross-entropy, mean over the batch.  dy[b, 0, :] = dlogits W_h^T, zero at
// every other position; the head gradients and the loss are added into
// gwh / gbh / loss.
// Every sum has one order, whatever the workgroups' order: the same inputs give
// the same bits (atomic adds in arrival order would not).
constexpr int HEAD_C = 16;        // maximum number of classes
constexpr int HEAD_NT = 1024;     // threads per workgroup (16 waves)
constexpr int HEAD_CHUNK = 256;   // samples per pass of head_ce_inplace_k

// rows 1 .. S-1 of every sequence of dY, by workgroup z of nz
template <typename T>
__device__ __forceinline__ void head_zero_rows(T* dy, int B, int S, int d, int z, int nz, bool nt) {
  const int vpr = d * (int)sizeof(T) / 16;  // 16-B vectors per row
  const long nvec = (long)B * (S - 1) * vpr;
  for (long v = (long)z * HEAD_NT + threadIdx.x; v < nvec; v += (long)nz * HEAD_NT) {
    const long rr = v / vpr;
    const long r = (rr / (S - 1)) * S + 1 + rr % (S - 1);
    st16(reinterpret_cast<uint4*>(dy + r * d) + v % vpr, zero_frag(), nt);
  }
}

// per-lane partial logits of K rows over features 8 (lane + 64 j)
template <typename T, int CN, int K>
__device__ __forceinline__ void head_dot(const T* const (&yr)[K], const float* wh, int d, int C, int lane,
                                         float (&lg)[K][CN]) {
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int c = 0; c < CN; ++c) lg[k][c] = 0.f;
  for (int v = lane; v < d / 8; v += 64) {
    float yv[K][8];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      if constexpr (std::is_same_v<T, bf16>) {
        unpack_frag(ld_frag(yr[k] + 8 * v), yv[k]);
      } else {
        const float4 q0 = reinterpret_cast<const float4*>(yr[k])[2 * v];
        const float4 q1 = reinterpret_cast<const float4*>(yr[k])[2 * v + 1];
        yv[k][0] = q0.x; yv[k][1] = q0.y; yv[k][2] = q0.z; yv[k][3] = q0.w;
        yv[k][4] = q1.x; yv[k][5] = q1.y; yv[k][6] = q1.z; yv[k][7] = q1.w;
      }
    }
    const float* wr = wh + (long)8 * v * C;
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int c = 0; c < CN; ++c)
        if (c < C) {
          const float wc = wr[e * C + c];
#pragma unroll
          for (int k = 0; k < K; ++k) lg[k][c] += yv[k][e] * wc;
        }
  }
}

// from the partial logits of one row: d loss / d logits (0 past C) in lg on
// every lane, the row's share of the mean loss returned
template <int CN>
__device__ __forceinline__ float head_softmax(float (&lg)[CN], const float* bh, int C, int lab, int B) {
  float mx = -INFINITY;
#pragma unroll
  for (int c = 0; c < CN; ++c)
    if (c < C) {
      lg[c] = wave_sum(lg[c]) + bh[c];
      mx = fmaxf(mx, lg[c]);
    }
  float se = 0.f, ll = 0.f;
#pragma unroll
  for (int c = 0; c < CN; ++c)
    if (c < C) {
      se += __expf(lg[c] - mx);
      if (c == lab) ll = lg[c];
    }
#pragma unroll
  for (int c = 0; c < CN; ++c)
    lg[c] = c < C ? (__expf(lg[c] - mx) / se - (c == lab ? 1.f : 0.f)) / (float)B : 0.f;
  return -(ll - mx - __logf(se)) / (float)B;
}

// Two classes: the first nf workgroups take HEAD_F features each, the others zero rows.  A
// wave owns every 16th sample: it forms that sample's logits from the whole row
// (every feature workgroup does so again: the rows are small and in the cache),
// then its lanes, one feature each, write dY and add to the W_h gradient, so
// nothing waits on another wave until the sums over the waves, in wave order,
// at the end.  What the end adds to is loaded at the start.  Bound by latency
// (one round trip for the rows, one launch): B 32, S 128, d 768 bf16 10.4 -> 5.9
// us, where one workgroup went through all features after a barrier.
constexpr int HEAD_F = 64;  // features per workgroup: one per lane
template <typename T>
__global__ __launch_bounds__(HEAD_NT) void head_ce2_k(const T* y, int B, int S, int d, const float* wh,
                                                      const float* bh, const int* labels, T* dy, float* gwh,
                                                      float* gbh, float* loss, int nf) {
  constexpr int C = 2, CN = 2;
  if ((int)blockIdx.x >= nf) {
    head_zero_rows(dy, B, S, d, (int)blockIdx.x - nf, (int)gridDim.x - nf,
                   stream_out((long)B * S * d * (long)sizeof(T)));
    return;
  }
  constexpr int NW = HEAD_NT / 64, PAIR = 2;
  __shared__ float red[NW][HEAD_F][CN];
  __shared__ float redb[NW][CN + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = threadIdx.x;
  const int f0 = blockIdx.x * HEAD_F, f = min(f0 + lane, d - 1);
  const bool fv = f0 + lane < d;
  const bool gv = t < HEAD_F * C && f0 * C + t < d * C, first = blockIdx.x == 0;
  const float gold = gv ? gwh[(long)f0 * C + t] : 0.f;
  const float bold = first && t < C ? gbh[t] : 0.f, lold = first && t == 0 && loss ? *loss : 0.f;
  float wv[CN], gacc[CN], bacc[CN], lacc = 0.f;
#pragma unroll
  for (int c = 0; c < CN; ++c) {
    wv[c] = wh[(long)f * C + c];
    gacc[c] = bacc[c] = 0.f;
  }
  for (int sm = wave; sm < B; sm += PAIR * NW) {
    const T* yr[PAIR];
    float yf[PAIR], lg[PAIR][CN];
    int lab[PAIR];
#pragma unroll
    for (int k = 0; k < PAIR; ++k) {
      const int smk = min(sm + k * NW, B - 1);
      yr[k] = y + (long)smk * S * d;
      yf[k] = St<T>::ld(yr[k], f);
      lab[k] = labels[smk];
    }
    head_dot<T, CN, PAIR>(yr, wh, d, C, lane, lg);
#pragma unroll
    for (int k = 0; k < PAIR; ++k) {
      if (sm + k * NW >= B) break;  // wave-uniform
      lacc += head_softmax<CN>(lg[k], bh, C, lab[k], B);
      float g = 0.f;
#pragma unroll
      for (int c = 0; c < CN; ++c) {
        gacc[c] += yf[k] * lg[k][c];
        bacc[c] += lg[k][c];
        g += lg[k][c] * wv[c];
      }
      if (fv) St<T>::st_nt(dy, (long)(sm + k * NW) * S * d + f, g);
    }
  }
#pragma unroll
  for (int c = 0; c < CN; ++c) red[wave][lane][c] = gacc[c];
  if (first && lane == 0) {
#pragma unroll
    for (int c = 0; c < CN; ++c) redb[wave][c] = bacc[c];
    redb[wave][CN] = lacc;
  }
  __syncthreads();
  if (gv) {
    float g = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) g += red[w][t / C][t % C];
    gwh[(long)f0 * C + t] = gold + g;
  }
  if (first && t < C) {
    float b = 0.f, l = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      b += redb[w][t];
      l += redb[w][CN];
    }
    gbh[t] = bold + b;
    if (t == 0 && loss) *loss = lold + l;
  }
}

// Up to 16 classes, the same division of the features.  The logits of 16 samples
// at a time are one 16x16 tile of MFMA 16x16x4 f32 (classes x samples), its K, the
// features, dealt to the 16 waves in blocks of 16; the waves' sums are added in
// LDS, 16 lanes share a sample for the softmax, then wave = sample and lane =
// feature as above.  One wave per sample read all of W_h for each, at a
// 512-B lane stride: B 128, S 16, d 4096, 16 classes 3947 -> 96 us, B 8,
// S 512, d 2048, 3 classes 35.5 -> 10.4 us.
template <typename T>
__global__ __launch_bounds__(HEAD_NT) void head_ce_many_k(const T* y, int B, int S, int d, const float* wh,
                                                          const float* bh, int C, const int* labels, T* dy,
                                                          float* gwh, float* gbh, float* loss, int nf) {
  if ((int)blockIdx.x >= nf) {
    head_zero_rows(dy, B, S, d, (int)blockIdx.x - nf, (int)gridDim.x - nf,
                   stream_out((long)B * S * d * (long)sizeof(T)));
    return;
  }
  constexpr int NW = HEAD_NT / 64, CN = HEAD_C;
  static_assert(NW == 16 && CN == 16, "16 samples x 16 classes, one sample per wave");
  __shared__ float part[NW][CN][17];
  __shared__ float sdl[NW][CN];
  __shared__ float sls[NW];
  __shared__ float red[NW][HEAD_F][CN];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = threadIdx.x, l16 = lane & 15, grp = lane >> 4;
  const int f0 = blockIdx.x * HEAD_F, f = min(f0 + lane, d - 1);
  const bool fv = f0 + lane < d;
  const bool gv = t < HEAD_F * C && f0 * C + t < d * C, first = blockIdx.x == 0;
  const float gold = gv ? gwh[(long)f0 * C + t] : 0.f;
  const float bold = first && t < C ? gbh[t] : 0.f, lold = first && t == 0 && loss ? *loss : 0.f;
  float wv[CN], gacc[CN], bacc = 0.f, lacc = 0.f;
#pragma unroll
  for (int c = 0; c < CN; ++c) {
    wv[c] = c < C ? wh[(long)f * C + c] : 0.f;
    gacc[c] = 0.f;
  }
  const int cls = min(l16, C - 1);
  for (int b0 = 0; b0 < B; b0 += NW) {
    const float yf = St<T>::ld(y, (long)min(b0 + wave, B - 1) * S * d + f);
    // samples past the batch read its last row, features past d the row's first: masked
    const T* yr = y + (long)min(b0 + l16, B - 1) * S * d;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int kb = wave * 16; kb < d; kb += 16 * NW) {
      const bool in = kb + 4 * grp < d;  // d is a multiple of 8: pieces of 4 are whole or absent
      const int k = in ? kb + 4 * grp : 0;
      float yv[4], w[4];
      St<T>::ld4(yr, k, yv);
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = wh[(long)(k + e) * C + cls];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(in && l16 < C ? w[e] : 0.f, in ? yv[e] : 0.f, acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave][4 * grp + r][l16] = acc[r];  // [class][sample]
    __syncthreads();
    if (t < NW * CN) {
      const int sm = t / CN, c = t % CN, lab = labels[min(b0 + sm, B - 1)];
      float lg = c < C ? bh[c] : 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) lg += part[w][c][sm];
      float mx = c < C ? lg : -INFINITY;
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
      const float e = c < C ? __expf(lg - mx) : 0.f;
      float se = e, ll = c == lab ? lg : 0.f;
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) {
        se += __shfl_xor(se, o, 64);
        ll += __shfl_xor(ll, o, 64);
      }
      const bool sv = b0 + sm < B && c < C;
      sdl[sm][c] = sv ? (e / se - (c == lab ? 1.f : 0.f)) / (float)B : 0.f;
      if (c == 0) sls[sm] = sv ? -(ll - mx - __logf(se)) / (float)B : 0.f;
    }
    __syncthreads();
    float g = 0.f;
#pragma unroll
    for (int c = 0; c < CN; ++c) {
      const float dl = sdl[wave][c];
      gacc[c] += yf * dl;
      g += dl * wv[c];
    }
    if (fv && b0 + wave < B) St<T>::st_nt(dy, (long)(b0 + wave) * S * d + f, g);
    if (first && t < C)
#pragma unroll
      for (int sm = 0; sm < NW; ++sm) {
        bacc += sdl[sm][t];
        lacc += sls[sm];
      }
  }
#pragma unroll
  for (int c = 0; c < CN; ++c) red[wave][lane][c] = gacc[c];
  __syncthreads();
  if (gv) {
    float g = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) g += red[w][t / C][t % C];
    gwh[(long)f0 * C + t] = gold + g;
  }
  if (first && t < C) gbh[t] = bold + bacc;
  if (first && t == 0 && loss) *loss = lold + lacc;
}

// dY in the place of y: one workgroup for all features.  Samples go in chunks of
// HEAD_CHUNK: one wave per sample for the logits, the softmax and the loss (into
// LDS), then, once the logits of the whole chunk are formed, one thread per
// feature (in blocks of HEAD_NT features) for the dY rows and the W_h gradient, so
// that a row is overwritten only after its last use; thread c for the bias
// gradient of class c and thread 0 for the loss.  The other workgroups zero rows
// 1..S-1 of every sequence.
template <typename T, int CN>  // CN: class count bound, compile time (the loops over classes unroll)
__global__ __launch_bounds__(HEAD_NT) void head_ce_inplace_k(const T* y, int B, int S, int d, const float* wh,
                                                     const float* bh, int C_, const int* labels, T* dy, float* gwh,
                                                     float* gbh, float* loss) {
  // the two-class instantiation runs only with C == 2: a compile-time class count leaves
  // no class guard around a load, so the loads of a row go out together
  const int C = CN == 2 ? 2 : C_;
  const bool nt = stream_out((long)B * S * d * (long)sizeof(T));  // dY streamed (common.h)
  if (blockIdx.x > 0) {
    head_zero_rows(dy, B, S, d, (int)blockIdx.x - 1, (int)gridDim.x - 1, nt);
    return;
  }
  constexpr int NW = HEAD_NT / 64;
  __shared__ float sdl[HEAD_CHUNK][CN];
  __shared__ float sls[HEAD_CHUNK];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = threadIdx.x;
  // logits, softmax and loss of samples b0 .. b0+nb-1 into sdl / sls, one wave each
  // samples per wave pass: two for the two-class head, so that both rows'
  // loads are in flight together (the second clamped); one for up to 16
  // classes, whose logits take the registers
  constexpr int PAIR = CN <= 4 ? 2 : 1;
  auto logits = [&](int b0, int nb) {
    for (int sm = wave; sm < nb; sm += PAIR * NW) {
      int smk[PAIR];
      const T* yr[PAIR];
#pragma unroll
      for (int k = 0; k < PAIR; ++k) {
        smk[k] = min(sm + k * NW, nb - 1);
        yr[k] = y + (long)(b0 + smk[k]) * S * d;
      }
      float lg[PAIR][CN];
      head_dot<T, CN, PAIR>(yr, wh, d, C, lane, lg);
#pragma unroll
      for (int k = 0; k < PAIR; ++k) {
        if (sm + k * NW >= nb) break;  // wave-uniform
        const float l = head_softmax<CN>(lg[k], bh, C, labels[b0 + smk[k]], B);
        if (lane == 0) {
          sls[smk[k]] = l;
#pragma unroll
          for (int c = 0; c < CN; ++c) sdl[smk[k]][c] = lg[k][c];
        }
      }
    }
  };
  float bacc = 0.f, lacc = 0.f;
  for (int b0 = 0; b0 < B; b0 += HEAD_CHUNK) {
    const int nb = min(HEAD_CHUNK, B - b0);
    if (b0 > 0) __syncthreads();  // every thread is done with the last chunk's sdl / sls
    logits(b0, nb);
    __syncthreads();
    for (int i = t; i < d; i += HEAD_NT) {
      float wv[CN], gacc[CN];
#pragma unroll
      for (int c = 0; c < CN; ++c) {
        wv[c] = c < C ? wh[(long)i * C + c] : 0.f;
        gacc[c] = 0.f;
      }
      // dY row and the W_h gradient of feature i (thread = feature), the samples in
      // order; UNR samples' loads in flight at once (clamped, masked after)
      constexpr int UNR = CN <= 4 ? 8 : 4;
      for (int sm0 = 0; sm0 < nb; sm0 += UNR) {
        float yv[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) yv[u] = St<T>::ld(y, (long)(b0 + min(sm0 + u, nb - 1)) * S * d + i);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const int sm = sm0 + u;
          if (sm >= nb) break;
          float g = 0.f;
#pragma unroll
          for (int c = 0; c < CN; ++c)
            if (c < C) {
              gacc[c] += yv[u] * sdl[sm][c];
              g += sdl[sm][c] * wv[c];
            }
          St<T>::st_nt(dy, (long)(b0 + sm) * S * d + i, g);
        }
      }
#pragma unroll
      for (int c = 0; c < CN; ++c)
        if (c < C) gwh[(long)i * C + c] += gacc[c];  // chunk by chunk, by this thread alone
    }
    if (t < C)
      for (int sm = 0; sm < nb; ++sm) bacc += sdl[sm][t];
    if (t == 0)
      for (int sm = 0; sm < nb; ++sm) lacc += sls[sm];
  }
  if (t < C) gbh[t] += bacc;
  if (t == 0 && loss) *loss += lacc;
}

// dY may be in the place of y, or clear of the rows of y that are read (position 0 of
// each sequence); otherwise some would be overwritten before their logits are formed
bool head_dy_ok(const void* y, const void* dy, int B, int S, size_t row) {
  if (y == dy) return true;
  const uintptr_t py = reinterpret_cast<uintptr_t>(y), pd = reinterpret_cast<uintptr_t>(dy);
  const uintptr_t step = (uintptr_t)S * row, end = pd + (uintptr_t)B * step;
  // the first of those rows that ends past dY's start
  const uintptr_t b = pd < py + row ? 0 : (pd - py - row) / step + 1;
  return b >= (uintptr_t)B || py + b * step >= end;
}

hipError_t launch_head_ce(int dtype, const void* y, int B, int S, int d, const float* wh, const float* bh,
                          int C, const int* labels, void* dy, float* gwh, float* gbh, float* loss,
                          hipStream_t s) {
  if (!y || !wh || !bh || !labels || !dy || !gwh || !gbh || B <= 0 || S <= 0 || d <= 0 || C < 1 || C > HEAD_C)
    return hipErrorInvalidValue;
  const size_t es = dtype == DT_BF16 ? 2 : 4;
  // rows move as 16-B vectors: d a multiple of 8, y, dy and w_h 16-B aligned
  if (d % 8 || (d * es) % 16 ||
      (reinterpret_cast<uintptr_t>(dy) | reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(wh)) & 15u)
    return hipErrorInvalidValue;
  const long nvec = (long)B * (S - 1) * (long)(d * es / 16);
  const int nz = (int)std::min<long>(255, (nvec + HEAD_NT - 1) / HEAD_NT);
  if (!head_dy_ok(y, dy, B, S, d * es)) return hipErrorInvalidValue;
  const bool inplace = y == dy;
  const int nf = inplace ? 1 : (d + HEAD_F - 1) / HEAD_F;
  const dim3 grid(nf + nz), block(HEAD_NT);
  auto go = [&](auto T0) {
    using T = decltype(T0);
    const T* yt = static_cast<const T*>(y);
    T* dt = static_cast<T*>(dy);
    if (inplace && C == 2)
      RG_LAUNCH((head_ce_inplace_k<T, 2>), grid, block, 0, s, yt, B, S, d, wh, bh, C, labels, dt, gwh, gbh, loss);
    else if (inplace)
      RG_LAUNCH((head_ce_inplace_k<T, HEAD_C>), grid, block, 0, s, yt, B, S, d, wh, bh, C, labels, dt, gwh, gbh,
                loss);
    else if (C == 2)
      RG_LAUNCH((head_ce2_k<T>), grid, block, 0, s, yt, B, S, d, wh, bh, labels, dt, gwh, gbh, loss, nf);
    else
      RG_LAUNCH((head_ce_many_k<T>), grid, block, 0, s, yt, B, S, d, wh, bh, C, labels, dt, gwh, gbh, loss, nf);
  };
  if (dtype == DT_BF16) go(bf16{});
  else go(float{});
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void sgd_f32_k(float* w, float* g, long n, float lr) {
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
    w[i] -= lr * g[i];
    g[i] = 0.f;
  }
}

hipError_t launch_sgd_f32(float* w, float* g, long n, float lr, hipStream_t s) {
  if (!w || !g || n <= 0) return hipErrorInvalidValue;
  const long nb = (n + 255) / 256;
  RG_LAUNCH(sgd_f32_k, dim3((unsigned)(nb < 1024 ? nb : 1024)), dim3(256), 0, s, w, g, n, lr);
  return hipGetLastError();
}

}  // namespace rg
