// pack.hip -- moe_quant_pack: group-wise asymmetric uniform quantization of
// fp32 rows and packing of the codes into 32-bit words; moe_requant_channels:
// the same quantizer applied to cached 16-bit channels, written into the
// 8-bit copy slots the FFN reads.
//
// Sec. IV-A (each expert quantized uniformly at its precision), Sec. V-B
// (several low-bit codes loaded as one 32-bit word) and Sec. IV-B
// (requantization of the cached channels for a new dataset).  The quantizer and the
// word layout are defined in moe_quant.h; parameter math is binary64, which
// gfx950 rounds exactly as IEEE requires, so the codes are reproducible bit
// for bit on any IEEE host.
#include <algorithm>

#include "common.hpp"

namespace moe {
namespace {

// Smallest binary16 >= s for a finite s > 0, by truncating the binary64
// significand and bumping the last kept bit when anything was cut off.
// Returns 0x7C00 (+inf) past 65504.
__device__ uint32_t fp16_ceil_bits(double s) {
  const uint64_t b = static_cast<uint64_t>(__double_as_longlong(s));
  const int e = static_cast<int>((b >> 52) & 0x7FF) - 1023;
  const uint64_t frac = b & ((1ull << 52) - 1);
  if (e < -24) return 1u;  // below the smallest subnormal 2^-24
  if (e < -14) {           // subnormal grid k * 2^-24, k = ceil(s * 2^24)
    const uint64_t full = (1ull << 52) | frac;
    const int sh = 52 - (e + 24);
    uint64_t k = full >> sh;
    if (full & ((1ull << sh) - 1)) k++;
    return static_cast<uint32_t>(k);  // k == 1024 is the pattern of 2^-14
  }
  if (e > 15) return 0x7C00u;
  uint32_t h = static_cast<uint32_t>(((e + 15) << 10) | (frac >> 42));
  if (frac & ((1ull << 42) - 1)) h++;  // may carry into the exponent, up to +inf
  return h;
}

// Value of an fp16 bit pattern as binary64 (exact).
__device__ double fp16_to_f64(uint32_t h) { return static_cast<double>(fp16_bits_to_f32(h)); }

// binary16 pattern of an integer 0 <= z <= 255 (exact).
__device__ uint32_t fp16_of_small_int(int z) {
  return __builtin_bit_cast(uint16_t, static_cast<_Float16>(static_cast<float>(z)));
}

// Bit position of local code i in a word of the b-bit half-split order.
__device__ __forceinline__ int hs_pos(int i, int b) { return (i >> 1) * b + 16 * (i & 1); }

// A group's range -> {scale, zero}: s = (mx - mn) / qmax, rounded up to
// binary16 (1.0 for an all-zero group), z = rint(-mn / s16).
struct Scale {
  uint32_t sb;   // binary16 pattern of the scale
  double sf;     // its value
  int z;
};

__device__ __forceinline__ Scale group_scale(double mn, double mx, int qmax) {
  Scale r;
  const double s = (mx - mn) / static_cast<double>(qmax);
  r.sb = (s == 0.0) ? 0x3C00u : fp16_ceil_bits(s);
  r.sf = fp16_to_f64(r.sb);
  const int z = static_cast<int>(rint(-mn / r.sf));
  r.z = z < 0 ? 0 : z;
  return r;
}

// The code of one value, clamp(rint(v / s) + z, 0, qmax) with the quotient in
// binary64.
__device__ __forceinline__ uint32_t code_f64(double v, const Scale& sc, int qmax) {
  double t = rint(v / sc.sf) + static_cast<double>(sc.z);
  t = t < 0.0 ? 0.0 : (t > static_cast<double>(qmax) ? static_cast<double>(qmax) : t);
  return static_cast<uint32_t>(t);
}

// The codes of N values of one group, the same integers as code_f64 mostly
// without its division: t = v * fl32(1/s) is within 2^-22 relative of v / s
// (two roundings of 2^-24 each), and |v / s| <= qmax because s >= (mx - mn) /
// qmax, so where t is more than qmax * 2^-21 away from every half integer,
// rint(t) is rint(v / s).  The values nearer to one (about one in 10^5 at 4
// bits, in 10^4 at 8), and NaN and infinities, take the division.
template <int N>
__device__ __forceinline__ void group_codes(const float (&v)[N], const Scale& sc, int qmax, uint32_t (&q)[N]) {
  const float rs = static_cast<float>(1.0 / sc.sf);
  const float edge = 0.5f - static_cast<float>(qmax) * 0x1p-21f;
  bool sure = true;
#pragma unroll
  for (int i = 0; i < N; i++) {
    const float t = v[i] * rs;
    const float n = rintf(t);
    sure = sure && __builtin_fabsf(t - n) < edge;   // false for NaN
    q[i] = static_cast<uint32_t>(min(max(static_cast<int>(n) + sc.z, 0), qmax));
  }
  if (!sure) {
#pragma unroll
    for (int i = 0; i < N; i++) q[i] = code_f64(static_cast<double>(v[i]), sc, qmax);
  }
}

// fp32 vector of any 4-byte alignment (rows of w may start anywhere)
typedef float f32x4a4 __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kPackRows = 16;    // most list rows of a workgroup
constexpr int kPackCols = 2048;  // most columns of a workgroup

// Rows per workgroup: 16, or fewer (down to 2) while that leaves less than
// four workgroups per compute unit of a full chip.
int pack_rows(int64_t n, int64_t K) {
  int rpw = kPackRows;
  while (rpw > 2 && cdiv(n, rpw) * cdiv(K, kPackCols) < 1024) rpw /= 2;
  return rpw;
}

// A grid holds fewer than 2^32 threads along x (the row blocks) and 65536 blocks
// along y (the column tiles): longer row lists and wider rows take several
// launches.  launch(i, m, c, k): list rows [i, i + m), columns [c, c + k).
constexpr int64_t kPackGridX = (int64_t{1} << 24) - 1;
constexpr int64_t kPackGridY = 32768;

template <typename F>
void pack_launches(int64_t n, int rpw, int64_t K, F launch) {
  for (int64_t c = 0; c < K; c += kPackGridY * kPackCols)
    for (int64_t i = 0; i < n; i += kPackGridX * rpw) {
      const int m = static_cast<int>(std::min(n - i, kPackGridX * rpw));
      const int k = static_cast<int>(std::min(K - c, kPackGridY * kPackCols));
      launch(i, m, c, k, dim3(static_cast<unsigned>(cdiv(m, rpw)), static_cast<unsigned>(cdiv(k, kPackCols))));
    }
}

// Quantize and pack rpw list rows x up to kPackCols columns per workgroup.
// Bound by the fp32 reads.  The tile's 8-weight items run over the threads row
// after row (a row of K columns holds a whole number of groups, so a group is
// 16 (or 8) neighbouring lanes at any K); a lane loads its 8 weights as two
// 16-byte loads, the range is reduced across the group's lanes, and every code
// word is put together from the lane's own codes or those of its pair or
// quad.  Two items per thread are in flight per step.  The {scale, zero}
// words go through LDS so that a group's words of 16 rows leave together (64
// bytes where they are row-contiguous).  Quantizing a 14336 x 4096 matrix at 4
// bits takes 62 us (4.2 TB/s of the 266 MB read and written, a copy 4.8)
// against 2040 us for one thread per (row, group), whose loads were 16 KB
// apart across lanes and which divided in binary64 once per weight.
template <int B, int GR>
__global__ void __launch_bounds__(256)
pack_kernel(const float* __restrict__ w, int64_t ld_w, int K, const int32_t* __restrict__ rows, int n, int rpw,
            uint32_t* __restrict__ codes, int64_t ld_codes, uint32_t* __restrict__ sz, int64_t sz_rs,
            int64_t sz_gs, int32_t* status) {
  constexpr int kLanes = GR / 8;   // lanes of a group
  constexpr int kGroups = kPackCols / GR;
  constexpr int qmax = (1 << (B & 15)) - 1;
  __shared__ uint32_t szl[kGroups][kPackRows];
  const int tid = threadIdx.x, lane = tid & 63;
  const int c0 = blockIdx.y * kPackCols;
  const int c8 = min(kPackCols, K - c0) / 8;   // items per row of the tile
  const int i0 = blockIdx.x * rpw;
  const int nr = min(rpw, n - i0);
  auto load = [&](float (&v)[8], int it) {
    const bool on = it < nr * c8;   // the same for all lanes of a group
    const int i = on ? it / c8 : 0;
    const int64_t r = on ? (rows ? static_cast<int64_t>(rows[i0 + i]) : i0 + i) : 0;
    const f32x4a4* p = reinterpret_cast<const f32x4a4*>(w + r * ld_w + c0 + 8 * (it - i * c8));
    f32x4a4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
    if (on) {
      a = p[0];
      b = p[1];
    }
#pragma unroll
    for (int c = 0; c < 4; c++) {
      v[c] = a[c];
      v[4 + c] = b[c];
    }
  };
  auto emit = [&](const float (&v)[8], int it) {
    const bool on = it < nr * c8;
    const int i = on ? it / c8 : 0;
    const int lc = 8 * (it - i * c8);   // column within the tile
    const int col = c0 + lc;
    const bool lead = on && lc % GR == 0;
    uint32_t* out = codes + static_cast<int64_t>(i0 + i) * ld_codes;
    if constexpr (B == 16) {   // unquantized: the bf16 value of each weight, scale 1 and zero 0
      u32x4 o;
#pragma unroll
      for (int c = 0; c < 4; c++) o[c] = bf16_rne(v[2 * c]) | (bf16_rne(v[2 * c + 1]) << 16);
      if (on) *reinterpret_cast<u32x4*>(out + col / 2) = o;
      if (lead) szl[lc / GR][i] = 0x3C00u;
      return;
    }
    float mn = 0.f, mx = 0.f;   // (a NaN leaves both as they are)
#pragma unroll
    for (int c = 0; c < 8; c++) {
      mn = v[c] < mn ? v[c] : mn;
      mx = v[c] > mx ? v[c] : mx;
    }
#pragma unroll
    for (int m = 1; m < kLanes; m <<= 1) {
      const float a = __shfl_xor(mn, m), b = __shfl_xor(mx, m);
      mn = a < mn ? a : mn;
      mx = b > mx ? b : mx;
    }
    const Scale sc = group_scale(static_cast<double>(mn), static_cast<double>(mx), qmax);
    if (lead) {
      szl[lc / GR][i] = sc.sb | (fp16_of_small_int(sc.z) << 16);
      if (sc.sb == 0x7C00u && status) *status = MOE_ERR_RANGE;
    }
    uint32_t q[8];
    group_codes<8>(v, sc, qmax, q);
    if constexpr (B == 8) {   // two words of four codes
      u32x2 o = {0u, 0u};
#pragma unroll
      for (int l = 0; l < 8; l++) o[l / 4] |= q[l] << hs_pos(l % 4, 8);
      if (on) *reinterpret_cast<u32x2*>(out + col / 4) = o;
    } else {
      // the low plane: 4 bits of 8 codes fill the lane's own word; 2 bits of
      // them are a byte of each half of a word shared by a pair of lanes
      constexpr int LB = (B == 4 || B == 6) ? 4 : 2;
      uint32_t lo = 0u, hi = 0u;
#pragma unroll
      for (int l = 0; l < 8; l++) lo |= (q[l] & ((1u << LB) - 1u)) << hs_pos(l, LB);
      if constexpr (LB == 2) lo = (lo << (8 * (lane & 1))) | (__shfl_xor(lo, 1) << (8 * (~lane & 1)));
      const int64_t blk = col / 32, q4 = lane & 3;   // 32-code block and the lane's place in it
      if constexpr (B == 4) {
        if (on) out[col / 8] = lo;
      } else if constexpr (B == 2) {
        if (on && (lane & 1) == 0) out[col / 16] = lo;
      } else if constexpr (B == 6) {   // words 0..3: low plane; 4, 5: bits 4..5 of the pairs
#pragma unroll
        for (int l = 0; l < 8; l++) hi |= (q[l] >> 4) << hs_pos(l, 2);
        hi = (hi << (8 * (lane & 1))) | (__shfl_xor(hi, 1) << (8 * (~lane & 1)));
        if (on) {
          out[6 * blk + q4] = lo;
          if ((lane & 1) == 0) out[6 * blk + 4 + q4 / 2] = hi;
        }
      } else {   // 3 bits, words 0, 1: low plane of the pairs; 2: bit 2 of the quad's 32 codes
#pragma unroll
        for (int l = 0; l < 8; l++) hi |= (q[l] >> 2) << hs_pos(l, 1);
        hi <<= 4 * q4;
        hi |= __shfl_xor(hi, 1);
        hi |= __shfl_xor(hi, 2);
        if (on) {
          if ((lane & 1) == 0) out[3 * blk + q4 / 2] = lo;
          if (q4 == 1) out[3 * blk + 2] = hi;
        }
      }
    }
  };
  for (int it = tid; it < nr * c8 + tid; it += 512) {   // uniform bound: lanes meet in the shuffles
    float a[8], b[8];
    load(a, it);
    load(b, it + 256);
    emit(a, it);
    emit(b, it + 256);
  }
  __syncthreads();
  for (int t = tid; t < kGroups * kPackRows; t += 256) {
    const int j = blockIdx.y * kGroups + t / kPackRows, i = t % kPackRows;
    if (j < K / GR && i < nr) sz[static_cast<int64_t>(i0 + i) * sz_rs + static_cast<int64_t>(j) * sz_gs] = szl[t / kPackRows][i];
  }
}

// Per-expert target precision of a requantization, passed by value
// (0 = the expert's slots are left as they are).
struct ExpertBits {
  uint8_t b[MOE_MAX_EXPERTS];
};

// words of any 4-byte alignment (all that is asked of the cache and of copy_codes)
typedef uint32_t u32x4a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32x2a4 __attribute__((ext_vector_type(2), aligned(4)));

// Requantize rpw copy slots x up to kPackCols columns per workgroup, in
// pack_kernel's shape: a lane takes 8 consecutive binary16 values of the
// cached row (one 16-byte load), a group is 16 (or 8) neighbouring lanes, and
// the quantizer is the same, so a row requantized at b bits carries exactly
// the codes moe_quant_pack gives for its binary16 values.  The b-bit codes are
// stored in the 8-bit copy format: each byte holds one code, bytes of a word in
// the 8-bit half-split order (two words per lane).  The 13112 cached channels
// of the Mixtral-shaped layer (8 experts, d 4096, d_ff 14336; 214 MB read and
// written in three launches) take 0.10 ms, against 0.23 ms with one wave per
// (slot, four groups) and the division in binary64 for every value.
template <int GR>
__global__ void __launch_bounds__(256)
requant_kernel(const uint16_t* __restrict__ cache, int64_t ld_cache, int K,
               const int32_t* __restrict__ hdr, int n_slots, int rpw, ExpertBits eb,
               uint32_t* __restrict__ codes, int64_t ld_codes, uint32_t* __restrict__ sz, int G,
               int32_t* status) {
  constexpr int kLanes = GR / 8;   // lanes of a group
  constexpr int kGroups = kPackCols / GR;
  __shared__ uint32_t szl[kPackRows][kGroups];
  __shared__ int32_t bit_of[kPackRows];   // precision of each slot's expert, 0: left alone
  const int tid = threadIdx.x;
  const int c0 = blockIdx.y * kPackCols;
  const int c8 = min(kPackCols, K - c0) / 8;   // items per row of the tile
  const int s0 = blockIdx.x * rpw;
  const int ns = min(rpw, n_slots - s0);
  if (tid < ns) bit_of[tid] = eb.b[hdr[2 * (s0 + tid)]];
  __syncthreads();
  // slot of an item: -1 past the tile and for slots left as they are (the
  // same for all lanes of a group)
  auto slot_of = [&](int it) {
    const int i = it < ns * c8 ? it / c8 : -1;
    return i >= 0 && bit_of[i] != 0 ? i : -1;
  };
  auto load = [&](int it) -> u32x4 {
    const int i = slot_of(it);
    u32x4 v = {0u, 0u, 0u, 0u};
    if (i >= 0)
      v = *reinterpret_cast<const u32x4a4*>(cache + static_cast<int64_t>(s0 + i) * ld_cache + c0 + 8 * (it - i * c8));
    return v;
  };
  auto emit = [&](const u32x4& raw, int it) {
    const int i = slot_of(it);
    const bool on = i >= 0;
    const int lc = on ? 8 * (it - i * c8) : 0;   // column within the tile
    const int qmax = on ? (1 << bit_of[i]) - 1 : 1;
    float v[8], mn = 0.f, mx = 0.f;
#pragma unroll
    for (int c = 0; c < 8; c++) {
      v[c] = fp16_bits_to_f32((c & 1) ? raw[c / 2] >> 16 : raw[c / 2] & 0xFFFFu);
      mn = v[c] < mn ? v[c] : mn;
      mx = v[c] > mx ? v[c] : mx;
    }
#pragma unroll
    for (int m = 1; m < kLanes; m <<= 1) {
      const float a = __shfl_xor(mn, m), b = __shfl_xor(mx, m);
      mn = a < mn ? a : mn;
      mx = b > mx ? b : mx;
    }
    const Scale sc = group_scale(static_cast<double>(mn), static_cast<double>(mx), qmax);
    uint32_t q[8];
    group_codes<8>(v, sc, qmax, q);
    u32x2 o = {0u, 0u};
#pragma unroll
    for (int l = 0; l < 8; l++) o[l / 4] |= q[l] << hs_pos(l % 4, 8);
    if (!on) return;
    *reinterpret_cast<u32x2a4*>(codes + static_cast<int64_t>(s0 + i) * ld_codes + (c0 + lc) / 4) = o;
    if (lc % GR == 0) {
      szl[i][lc / GR] = sc.sb | (fp16_of_small_int(sc.z) << 16);
      if (sc.sb == 0x7C00u && status) *status = MOE_ERR_RANGE;
    }
  };
  for (int it = tid; it < ns * c8 + tid; it += 1024) {   // uniform bound: lanes meet in the shuffles
    u32x4 raw[4];
#pragma unroll
    for (int u = 0; u < 4; u++) raw[u] = load(it + 256 * u);
#pragma unroll
    for (int u = 0; u < 4; u++) emit(raw[u], it + 256 * u);
  }
  __syncthreads();
  for (int t = tid; t < kGroups * ns; t += 256) {
    const int i = t / kGroups, j = blockIdx.y * kGroups + t % kGroups;
    if (j < K / GR && bit_of[i] != 0) sz[static_cast<int64_t>(s0 + i) * G + j] = szl[i][t % kGroups];
  }
}

}  // namespace
}  // namespace moe

extern "C" int moe_quant_pack(const float* w, int64_t ld_w, int32_t R, int32_t K,
                              int32_t bits, int32_t group, const int32_t* rows, int32_t n,
                              uint32_t* codes, int64_t ld_codes, uint32_t* sz,
                              int64_t sz_row_stride, int64_t sz_group_stride,
                              int32_t* status, void* stream) {
  using namespace moe;
  if (!valid_expert_bits(bits)) return MOE_ERR_BITS;
  if (!w || !codes || !sz || R <= 0 || K <= 0 || n < 0) return MOE_ERR_ARG;
  if (!(group == 64 || group == 128) || K % group || K % 32) return MOE_ERR_ARG;
  if ((bits == 3 || bits == 6) && group != 128) return MOE_ERR_ARG;
  if (ld_w < K || ld_codes < static_cast<int64_t>(K) * bits / 32) return MOE_ERR_ARG;
  if (!rows && n > R) return MOE_ERR_ARG;
  if (!aligned16(codes) || (ld_codes * 4) % 16) return MOE_ERR_ALIGN;
  if (n == 0) return MOE_OK;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int rpw = pack_rows(n, K);
  auto launch = [&](auto kernel) {
    pack_launches(n, rpw, K, [&](int64_t i, int m, int64_t c, int k, dim3 grid) {
      hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, (rows ? w : w + i * ld_w) + c, ld_w, k, rows ? rows + i : rows, m,
                         rpw, codes + i * ld_codes + c * bits / 32, ld_codes,
                         sz + i * sz_row_stride + c / group * sz_group_stride, sz_row_stride, sz_group_stride, status);
    });
  };
  if (group == 64) {
    switch (bits) {
      case 2: launch(pack_kernel<2, 64>); break;
      case 4: launch(pack_kernel<4, 64>); break;
      case 8: launch(pack_kernel<8, 64>); break;
      default: launch(pack_kernel<16, 64>); break;
    }
  } else {
    switch (bits) {
      case 2: launch(pack_kernel<2, 128>); break;
      case 3: launch(pack_kernel<3, 128>); break;
      case 4: launch(pack_kernel<4, 128>); break;
      case 6: launch(pack_kernel<6, 128>); break;
      case 8: launch(pack_kernel<8, 128>); break;
      default: launch(pack_kernel<16, 128>); break;
    }
  }
  return launch_status(s);
}

extern "C" int moe_requant_channels(moe_layer_t* L, int32_t kind, const uint16_t* cache,
                                    int64_t ld_cache, const int32_t* expert_bits,
                                    int32_t* status, void* stream) {
  using namespace moe;
  if (!L || kind < 0 || kind > 2 || !expert_bits) return MOE_ERR_ARG;
  const int E = L->n_experts;
  if (E <= 0 || E + L->n_shared > MOE_MAX_EXPERTS) return MOE_ERR_ARG;
  if (!(L->group == 64 || L->group == 128)) return MOE_ERR_ARG;
  const int K = kind == MOE_KIND_DOWN ? L->d_ff : L->d_model;
  if (K <= 0 || K % L->group || K % 128) return MOE_ERR_ARG;
  ExpertBits eb{};
  for (int e = 0; e < E; e++) {
    const int b = expert_bits[e];
    if (b != 0 && !valid_bits(b)) return MOE_ERR_BITS;
    eb.b[e] = static_cast<uint8_t>(b);
  }
  const moe_kind_desc_t& D = L->kind[kind];
  if (D.n_slots < 0) return MOE_ERR_ARG;
  if (D.n_slots == 0) return MOE_OK;
  if (!cache || ld_cache < K || (ld_cache % 2) || (reinterpret_cast<uintptr_t>(cache) & 3u))
    return MOE_ERR_ARG;
  if (!D.copy_codes || !D.copy_sz || !D.copy_hdr || !D.copy_hdr_host) return MOE_ERR_ARG;
  for (int sl = 0; sl < D.n_slots; sl++) {
    const int e = D.copy_hdr_host[2 * sl];
    if (e < 0 || e >= E) return MOE_ERR_SLOT;
  }
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int rpw = pack_rows(D.n_slots, K);
  auto launch = [&](auto kernel) {
    pack_launches(D.n_slots, rpw, K, [&](int64_t i, int m, int64_t c, int k, dim3 grid) {
      hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, cache + i * ld_cache + c, ld_cache, k, D.copy_hdr + 2 * i, m, rpw,
                         eb, const_cast<uint32_t*>(D.copy_codes) + i * code_row_words(K, 8) + c / 4, code_row_words(K, 8),
                         const_cast<uint32_t*>(D.copy_sz) + i * (K / L->group) + c / L->group, K / L->group, status);
    });
  };
  if (L->group == 64) launch(requant_kernel<64>);
  else launch(requant_kernel<128>);
  return launch_status(s);
}

extern "C" const char* moe_status_str(int status) {
  switch (status) {
    case MOE_OK: return "ok";
    case MOE_ERR_ARG: return "invalid argument";
    case MOE_ERR_BITS: return "bit-width not in {2,3,4,6,8} (or 16 where allowed)";
    case MOE_ERR_ALIGN: return "pointer or stride not 16-byte aligned";
    case MOE_ERR_WORKSPACE: return "workspace missing or too small";
    case MOE_ERR_SLOT: return "bad switch slot list";
    case MOE_ERR_RANGE: return "fp16 scale overflow";
    case MOE_ERR_HIP: return "HIP error";
    default: return "unknown status";
  }
}

extern "C" int64_t moe_code_row_words(int32_t K, int32_t bits) {
  if (!moe::valid_expert_bits(bits) || K <= 0 || K % 128) return 0;
  return moe::code_row_words(K, bits);
}
