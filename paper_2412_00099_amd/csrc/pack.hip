// Blob geometry, the canonical -> record-layout packer, and the synthetic-stack glue kernel.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gemv_common.h"

namespace moe {

BlobLayout blob_layout(int fmt, int hidden, int inter) {
  BlobLayout L{};
  const int64_t d = hidden, I = inter;
  int64_t tail_bytes = 0;
  switch (fmt) {
    case MOE_W_FP32:
      L.row_bytes = d * 4;
      L.rec_bytes = 3 * L.row_bytes;
      break;
    case MOE_W_BF16:
      L.row_bytes = d * 2;
      L.rec_bytes = 3 * L.row_bytes;
      break;
    case MOE_W_INT8_PC:  // tail: gate scales [I], up scales [I], down scales [d], fp16
      L.row_bytes = d;
      L.rec_bytes = 3 * L.row_bytes;
      tail_bytes = (2 * I + d) * 2;
      break;
    case MOE_W_INT4_G128:  // record carries its (gate, up) group scales; tail: down scales [I/128][d], fp16
      L.row_bytes = d / 2;
      L.rec_bytes = int4_record_bytes(d);
      tail_bytes = (I / 128) * d * 2;
      break;
    default: return L;
  }
  L.tail_offset = I * L.rec_bytes;
  L.total = (L.tail_offset + tail_bytes + 255) / 256 * 256;
  return L;
}

namespace {

// The packers are copies bound by HBM.  gate and up rows move as 16-byte chunks.  W_down is transposed: its columns
// become record rows.  A lane takes a block of CT columns x RT records, whose loads and stores are 8 to 16 bytes, and
// transposes it in registers; the lanes of a wavefront are laid out CL x RL over (columns, records) so that a load
// covers 64 to 128 bytes of each of its rows of W_down and a store as much of each record.  (One chunk of a record per
// thread, gathered element by element from as many rows, fetched a line per element: d = 2048, I = 1408 took 20 us in
// bf16 and 21.6 us in int4; now 7.2 us - 34.6 MB, 4.8 TB/s - and 4.3 us.)  Blocks 0 .. n_tr-1 transpose, the others
// copy; one launch.
constexpr int kPackBlock = 256;

// 16 bytes from / to memory that may be aligned to T only
template <bool ALIGNED, typename T>
__device__ __forceinline__ u32x4 ld16(const T *p) {
  if constexpr (ALIGNED) {
    return *reinterpret_cast<const u32x4 *>(p);
  } else {
    union { T e[16 / sizeof(T)]; u32x4 v; } u;
#pragma unroll
    for (int i = 0; i < (int)(16 / sizeof(T)); ++i) u.e[i] = p[i];
    return u.v;
  }
}
template <bool ALIGNED, typename T>
__device__ __forceinline__ void st16(T *p, const u32x4 &v) {
  if constexpr (ALIGNED) {
    *reinterpret_cast<u32x4 *>(p) = v;
  } else {
    union { T e[16 / sizeof(T)]; u32x4 v; } u;
    u.v = v;
#pragma unroll
    for (int i = 0; i < (int)(16 / sizeof(T)); ++i) p[i] = u.e[i];
  }
}

// gate and up rows (row_chunks 16-byte chunks each) into records of rec_elems elements; every word XORed with flip
template <bool ALIGNED, typename T>
__device__ __forceinline__ void copy_rows(const T *gate, const T *up, T *blob, int64_t I, int row_chunks, int64_t rec_elems,
                                          uint32_t flip, int block, int n_blocks) {
  constexpr int VEC = 16 / sizeof(T), PER = 4;
  const int64_t n = I * row_chunks;  // chunks of one matrix
  for (int64_t c0 = ((int64_t)block * kPackBlock) * PER + threadIdx.x; c0 < 2 * n; c0 += (int64_t)n_blocks * kPackBlock * PER) {
    u32x4 v[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int64_t c = c0 + j * kPackBlock;
      if (c < 2 * n) v[j] = ld16<ALIGNED>((c < n ? gate : up - n * VEC) + c * VEC);
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int64_t c = c0 + j * kPackBlock;
      if (c >= 2 * n) break;
      const int64_t m = c < n ? c : c - n, rec = m / row_chunks, k = m - rec * row_chunks;
      st16<ALIGNED>(blob + rec * rec_elems + ((c < n ? 0 : row_chunks) + k) * VEC, v[j] ^ flip);
    }
  }
}

// fp32 / bf16: a lane transposes VEC columns x VEC records
template <typename T, bool ALIGNED>
__global__ __launch_bounds__(kPackBlock) void pack_plain_kernel(const T *gate, const T *up, const T *down, T *blob, int d, int I,
                                                                int n_tr) {
  constexpr int VEC = 16 / sizeof(T);
  if ((int)blockIdx.x >= n_tr) {
    copy_rows<ALIGNED>(gate, up, blob, I, d / VEC, 3 * (int64_t)d, 0u, (int)blockIdx.x - n_tr, (int)gridDim.x - n_tr);
    return;
  }
  const int lane = threadIdx.x & 63, cb = lane & 7, rb = lane >> 3;
  const int tile = (int)blockIdx.x * (kPackBlock / 64) + (threadIdx.x >> 6), ct = d / (8 * VEC);
  const int col = (tile % ct * 8 + cb) * VEC;
  const int64_t rec = (int64_t)(tile / ct * 8 + rb) * VEC;
  if (rec >= I) return;
  const bool whole = ALIGNED && I % VEC == 0;  // every row of W_down starts on 16 bytes
  const int n = (int)min((int64_t)VEC, I - rec);
  T *o = blob + (rec * 3 + 2) * d + col;
  u32x4 in[VEC];
#pragma unroll
  for (int j = 0; j < VEC; ++j) {
    const T *q = down + (int64_t)(col + j) * I + rec;
    if (whole) {
      in[j] = *reinterpret_cast<const u32x4 *>(q);
    } else {
      union { T e[VEC]; u32x4 v; } u;
#pragma unroll
      for (int i = 0; i < VEC; ++i) u.e[i] = q[i < n ? i : 0];
      in[j] = u.v;
    }
  }
#pragma unroll
  for (int i = 0; i < VEC; ++i) {
    u32x4 out;
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int j = 0; j < 4; ++j) out[j] = in[j][i];
    } else {
      const uint32_t sel = (i & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
      for (int j = 0; j < 4; ++j) out[j] = __builtin_amdgcn_perm(in[2 * j + 1][i >> 1], in[2 * j][i >> 1], sel);
    }
    if (i < n) st16<ALIGNED>(o + (int64_t)i * 3 * d, out);
  }
}

// 4 x 4 bytes: r[i] byte j -> c[j] byte i
__device__ __forceinline__ void transpose4(const uint32_t (&r)[4], uint32_t (&c)[4]) {
  const uint32_t a0 = __builtin_amdgcn_perm(r[1], r[0], 0x05010400u), a1 = __builtin_amdgcn_perm(r[1], r[0], 0x07030602u);
  const uint32_t b0 = __builtin_amdgcn_perm(r[3], r[2], 0x05010400u), b1 = __builtin_amdgcn_perm(r[3], r[2], 0x07030602u);
  c[0] = __builtin_amdgcn_perm(b0, a0, 0x05040100u);
  c[1] = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
  c[2] = __builtin_amdgcn_perm(b1, a1, 0x05040100u);
  c[3] = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
}

// int8: values become offset-binary bytes (q + 128); scales go to the tail.  A lane transposes 16 columns x 8 records.
template <bool ALIGNED>
__global__ __launch_bounds__(kPackBlock) void pack_int8_kernel(const uint8_t *gate, const uint8_t *up, const uint8_t *down,
                                                               const uint16_t *gs, const uint16_t *us, const uint16_t *ds,
                                                               uint8_t *blob, int d, int I, int n_tr) {
  constexpr uint32_t kFlip = 0x80808080u;
  if ((int)blockIdx.x >= n_tr) {
    const int block = (int)blockIdx.x - n_tr, n_blocks = (int)gridDim.x - n_tr;
    uint16_t *tail = reinterpret_cast<uint16_t *>(blob + (int64_t)I * 3 * d);
    for (int64_t i = (int64_t)block * kPackBlock + threadIdx.x; i < 2 * (int64_t)I + d; i += (int64_t)n_blocks * kPackBlock)
      tail[i] = i < I ? gs[i] : i < 2 * (int64_t)I ? us[i - I] : ds[i - 2 * I];
    copy_rows<ALIGNED>(gate, up, blob, I, d / 16, 3 * (int64_t)d, kFlip, block, n_blocks);
    return;
  }
  const int lane = threadIdx.x & 63, cb = lane & 7, rb = lane >> 3;
  const int tile = (int)blockIdx.x * (kPackBlock / 64) + (threadIdx.x >> 6), ct = d / 128;
  const int col = (tile % ct * 8 + cb) * 16;
  const int64_t rec = (int64_t)(tile / ct * 8 + rb) * 8;  // (I is a multiple of 8)
  if (rec >= I) return;
  uint32_t in[16][2];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const uint8_t *q = down + (int64_t)(col + j) * I + rec;
    if constexpr (ALIGNED) {
      const u32x2 v = *reinterpret_cast<const u32x2 *>(q);
      in[j][0] = v.x;
      in[j][1] = v.y;
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        in[j][h] = (uint32_t)q[4 * h] | ((uint32_t)q[4 * h + 1] << 8) | ((uint32_t)q[4 * h + 2] << 16) | ((uint32_t)q[4 * h + 3] << 24);
    }
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {  // records 4 h .. + 4
    uint32_t c[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t r[4] = {in[4 * j][h], in[4 * j + 1][h], in[4 * j + 2][h], in[4 * j + 3][h]};
      uint32_t t[4];
      transpose4(r, t);
#pragma unroll
      for (int i = 0; i < 4; ++i) c[i][j] = t[i] ^ kFlip;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      st16<ALIGNED>(blob + ((rec + 4 * h + i) * 3 + 2) * d + col, u32x4{c[i][0], c[i][1], c[i][2], c[i][3]});
  }
}

// 8 x 8 nibbles in place: r[i] nibble j -> r[j] nibble i, by swapping off-diagonal blocks of S = 4, 2 and 1
template <int S>
__device__ __forceinline__ void swap_nibble_blocks(uint32_t (&r)[8]) {
  constexpr uint32_t mask = S == 4 ? 0x0000ffffu : S == 2 ? 0x00ff00ffu : 0x0f0f0f0fu;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (i & S) continue;
    const uint32_t x = ((r[i] >> (4 * S)) ^ r[i + S]) & mask;
    r[i + S] ^= x;
    r[i] ^= x << (4 * S);
  }
}
__device__ __forceinline__ void transpose_nibbles(uint32_t (&r)[8]) {
  swap_nibble_blocks<4>(r);
  swap_nibble_blocks<2>(r);
  swap_nibble_blocks<1>(r);
}

// int4: canonical bytes hold two nibbles (even column low).  A lane transposes 16 columns x 8 records of W_down; the
// record ends with its (gate, up) scale pairs, the down scales form the tail.
template <bool ALIGNED>
__global__ __launch_bounds__(kPackBlock) void pack_int4_kernel(const uint8_t *gate, const uint8_t *up, const uint8_t *down,
                                                               const uint16_t *gs, const uint16_t *us, const uint16_t *ds,
                                                               uint8_t *blob, int d, int I, int n_tr) {
  const int64_t row_bytes = d / 2, groups = d / 128, rec_bytes = int4_record_bytes(d);
  if ((int)blockIdx.x >= n_tr) {
    const int block = (int)blockIdx.x - n_tr, n_blocks = (int)gridDim.x - n_tr;
    const int64_t gid = (int64_t)block * kPackBlock + threadIdx.x, stride = (int64_t)n_blocks * kPackBlock;
    for (int64_t i = gid; i < (int64_t)I * groups; i += stride) {
      const int64_t rec = i / groups, g = i - rec * groups;
      uint16_t *o = reinterpret_cast<uint16_t *>(blob + rec * rec_bytes + 3 * row_bytes + g * 4);
      o[0] = gs[i];
      o[1] = us[i];
    }
    uint16_t *tail = reinterpret_cast<uint16_t *>(blob + (int64_t)I * rec_bytes);
    const int64_t rgroups = I / 128;
    for (int64_t i = gid; i < rgroups * d; i += stride) {
      const int64_t g = i / d, col = i - g * d;
      tail[i] = ds[col * rgroups + g];
    }
    copy_rows<ALIGNED>(gate, up, blob, I, (int)(row_bytes / 16), rec_bytes, 0u, block, n_blocks);
    return;
  }
  const int lane = threadIdx.x & 63, cb = lane & 7, rb = lane >> 3;
  const int tile = (int)blockIdx.x * (kPackBlock / 64) + (threadIdx.x >> 6), ct = d / 128;
  const int col = (tile % ct * 8 + cb) * 16;
  const int64_t rec = (int64_t)(tile / ct * 8 + rb) * 8;  // (I is a multiple of 128)
  if (rec >= I) return;
  const int64_t in_row = I / 2;
  uint32_t r[2][8];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const uint8_t *q = down + (col + j) * in_row + rec / 2;
    if constexpr (ALIGNED) r[j >> 3][j & 7] = *reinterpret_cast<const uint32_t *>(q);
    else r[j >> 3][j & 7] = (uint32_t)q[0] | ((uint32_t)q[1] << 8) | ((uint32_t)q[2] << 16) | ((uint32_t)q[3] << 24);
  }
  transpose_nibbles(r[0]);
  transpose_nibbles(r[1]);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    uint8_t *o = blob + (rec + i) * rec_bytes + 2 * row_bytes + col / 2;
    if constexpr (ALIGNED) {
      *reinterpret_cast<u32x2 *>(o) = u32x2{r[0][i], r[1][i]};
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        o[k] = (uint8_t)(r[0][i] >> (8 * k));
        o[4 + k] = (uint8_t)(r[1][i] >> (8 * k));
      }
    }
  }
}

// h = (carry ? h : 0) + y + perturb*a ; x = h / sqrt(mean(h^2) + 1e-6) in act_fmt.  One workgroup.
__global__ __launch_bounds__(1024) void residual_rmsnorm_kernel(float *h, const void *y, const float *a,
                                                                float perturb, int carry, void *x, int d,
                                                                int act_fmt) {
  __shared__ float part[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float ss = 0.f;
  for (int j = tid; j < d; j += blockDim.x) {
    float v = carry ? h[j] : 0.f;
    if (y) v += (act_fmt == MOE_A_BF16) ? __uint_as_float((uint32_t) static_cast<const uint16_t *>(y)[j] << 16)
                                        : static_cast<const float *>(y)[j];
    if (a) v = __builtin_fmaf(perturb, a[j], v);
    h[j] = v;
    ss = __builtin_fmaf(v, v, ss);
  }
  ss = wave_sum(ss);
  if (lane == 0) part[wave] = ss;
  __syncthreads();
  float tot = 0.f;
  for (int w = 0; w < (int)(blockDim.x >> 6); ++w) tot += part[w];
  const float scale = 1.0f / sqrtf(tot / (float)d + 1e-6f);
  for (int j = tid; j < d; j += blockDim.x) {
    const float v = h[j] * scale;
    if (act_fmt == MOE_A_BF16)
      static_cast<uint16_t *>(x)[j] = f32_to_bf16_rne(v);
    else
      static_cast<float *>(x)[j] = v;
  }
}

}  // namespace

hipError_t launch_pack(int fmt, int hidden, int inter, const void *gate, const void *up, const void *down,
                       const void *gs, const void *us, const void *ds, void *blob, hipStream_t s) {
  // transposing blocks: four wavefronts, each with a tile of (8 x columns per lane) x (8 x records per lane)
  int col_tile = 0, rec_tile = 0, per16 = 0;
  switch (fmt) {
    case MOE_W_FP32: col_tile = 32; rec_tile = 32; per16 = 4; break;
    case MOE_W_BF16: col_tile = 64; rec_tile = 64; per16 = 8; break;
    case MOE_W_INT8_PC: col_tile = 128; rec_tile = 64; per16 = 16; break;
    case MOE_W_INT4_G128: col_tile = 128; rec_tile = 64; per16 = 32; break;
    default: return hipErrorInvalidValue;
  }
  const int64_t tiles = (int64_t)(hidden / col_tile) * ((inter + rec_tile - 1) / rec_tile);
  const int64_t chunks = 2 * (int64_t)inter * hidden / per16;
  const int64_t n_tr = (tiles + 3) / 4, n_copy = std::min<int64_t>((chunks + 4 * kPackBlock - 1) / (4 * kPackBlock), 65536);
  if (n_tr + n_copy > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 g((uint32_t)(n_tr + n_copy)), b(kPackBlock);
  uintptr_t any = reinterpret_cast<uintptr_t>(gate) | reinterpret_cast<uintptr_t>(up) | reinterpret_cast<uintptr_t>(down) |
                  reinterpret_cast<uintptr_t>(blob);
  const bool aligned = any % 16 == 0;  // whatever the caller has; views into larger tensors may not be
  const auto run = [&](auto kernel, auto... args) { hipLaunchKernelGGL(kernel, g, b, 0, s, args..., hidden, inter, (int)n_tr); };
  const auto plain = [&](auto kernel, auto *t) {
    using T = std::remove_pointer_t<decltype(t)>;
    run(kernel, static_cast<const T *>(gate), static_cast<const T *>(up), static_cast<const T *>(down), static_cast<T *>(blob));
  };
  const auto quant = [&](auto kernel) {
    run(kernel, static_cast<const uint8_t *>(gate), static_cast<const uint8_t *>(up), static_cast<const uint8_t *>(down),
        static_cast<const uint16_t *>(gs), static_cast<const uint16_t *>(us), static_cast<const uint16_t *>(ds),
        static_cast<uint8_t *>(blob));
  };
  switch (fmt) {
    case MOE_W_FP32: plain(aligned ? pack_plain_kernel<float, true> : pack_plain_kernel<float, false>, (float *)nullptr); break;
    case MOE_W_BF16: plain(aligned ? pack_plain_kernel<uint16_t, true> : pack_plain_kernel<uint16_t, false>, (uint16_t *)nullptr); break;
    case MOE_W_INT8_PC: quant(aligned ? pack_int8_kernel<true> : pack_int8_kernel<false>); break;
    default: quant(aligned ? pack_int4_kernel<true> : pack_int4_kernel<false>);
  }
  return hipGetLastError();
}

hipError_t launch_residual_rmsnorm(float *h, const void *y, const float *a, float perturb, int carry, void *x,
                                   int hidden, int act_fmt, hipStream_t s) {
  hipLaunchKernelGGL(residual_rmsnorm_kernel, dim3(1), dim3(1024), 0, s, h, y, a, perturb, carry, x, hidden,
                     act_fmt);
  return hipGetLastError();
}

}  // namespace moe
