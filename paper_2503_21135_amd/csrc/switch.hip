// switch.hip -- moe_set_channel_switch: install a set of cached 8-bit copies.
//
// Sec. IV-B "Channel Weights Replacement based on Caching": a cached channel
// replaces the quantized channel whose (expert, channel) index it carries.
// Sec. V-A "Data Format in the Channel Cache": the expert and channel indexes
// are stored as headers of the cache entries so the target is found directly.
// Here the headers are scattered into a per-(expert, row) table (row_slot), so
// the FFN finds a row's source with one load; no weights move and nothing is
// requantized.  The visiting order of rows (order_gu / order_dn) is rebuilt
// as a stable partition by precision source, which keeps most 16-row tiles of
// the FFN uniform in bit-width.
#include <vector>

#include "common.hpp"

namespace moe {
namespace {

__global__ void __launch_bounds__(256) fill_kernel(int32_t* p, int64_t n, int32_t v) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void __launch_bounds__(256)
scatter_slots_kernel(const int32_t* __restrict__ list, int n, const int32_t* __restrict__ hdr,
                     int R, int32_t* __restrict__ row_slot) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int s = list[i];
  const int e = hdr[2 * s];
  const int r = hdr[2 * s + 1];
  row_slot[static_cast<int64_t>(e) * R + r] = s;
}

constexpr int kOrderWaves = 16;  // waves of the order workgroup

// One workgroup (16 waves) per routed expert.  Class of row i:
// bit 0 = row_slot_a[i] >= 0, bit 1 = row_slot_b[i] >= 0 (b may be NULL).
// order lists class 0 rows ascending, then class 1, 2, 3; class_cnt[4e + c]
// receives the size of class c.  Wave w takes the w-th run of the expert's
// rows: it counts its classes (64 rows per step, ballots), the 16 waves' counts
// are scanned once, and it places its rows in a second pass over the run --
// two barriers in all, where a barrier per 256 rows made the wide experts'
// launch a chain of 56 of them (8 experts of 14336
// rows: 64 -> 15 us; 64 experts of 1408 rows: 21 -> 5 us).
__global__ void __launch_bounds__(kOrderWaves * kWave)
order_kernel(const int32_t* __restrict__ rs_a, const int32_t* __restrict__ rs_b, int R,
             int32_t* __restrict__ order, int32_t* __restrict__ class_cnt) {
  __shared__ int wave_cnt[4][kOrderWaves];
  const int e = blockIdx.x;
  const int wv = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  rs_a += static_cast<int64_t>(e) * R;
  if (rs_b) rs_b += static_cast<int64_t>(e) * R;
  order += static_cast<int64_t>(e) * R;
  const int steps = (R + kOrderWaves * kWave - 1) / (kOrderWaves * kWave);
  const int r0 = wv * steps * kWave, r1 = min(r0 + steps * kWave, R);
  constexpr int U = 4;   // steps whose loads are issued together
  auto classes = [&](int base, int (&c)[U]) {
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int i = base + u * kWave + lane;
      const bool live = i < r1;
      const int a = live ? rs_a[i] : -1, b = (live && rs_b) ? rs_b[i] : -1;
      c[u] = live ? ((a >= 0 ? 1 : 0) | (b >= 0 ? 2 : 0)) : -1;
    }
  };
  int cnt[4] = {0, 0, 0, 0};
  for (int base = r0; base < r1; base += U * kWave) {
    int c[U];
    classes(base, c);
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int cc = 0; cc < 4; cc++) cnt[cc] += __popcll(__ballot(c[u] == cc));
  }
  if (lane < 4) wave_cnt[lane][wv] = lane == 0 ? cnt[0] : (lane == 1 ? cnt[1] : (lane == 2 ? cnt[2] : cnt[3]));
  __syncthreads();
  // first position of each class in this wave's run
  int pos[4], start = 0;
#pragma unroll
  for (int cc = 0; cc < 4; cc++) {
    int before = 0, total = 0;
#pragma unroll
    for (int w2 = 0; w2 < kOrderWaves; w2++) {
      const int v = wave_cnt[cc][w2];
      before += w2 < wv ? v : 0;
      total += v;
    }
    pos[cc] = start + before;
    start += total;
    if (threadIdx.x == 0) class_cnt[4 * e + cc] = total;
  }
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  for (int base = r0; base < r1; base += U * kWave) {
    int c[U];
    classes(base, c);
#pragma unroll
    for (int u = 0; u < U; u++)
#pragma unroll
      for (int cc = 0; cc < 4; cc++) {
        const uint64_t m = __ballot(c[u] == cc);
        if (c[u] == cc) order[pos[cc] + __popcll(m & below)] = base + u * kWave + lane;
        pos[cc] += __popcll(m);
      }
  }
}

int rows_of_kind(const moe_layer_t* L, int kind) {
  return kind == MOE_KIND_DOWN ? L->d_model : L->d_ff;
}

}  // namespace
}  // namespace moe

extern "C" int moe_set_channel_switch(moe_layer_t* L, int32_t kind, const int32_t* slots_on,
                                      int32_t n_on, void* stream) {
  using namespace moe;
  if (!L || L->n_experts <= 0 || L->d_model <= 0 || L->d_ff <= 0) return MOE_ERR_ARG;
  if (!L->order_gu || !L->order_dn || !L->class_cnt) return MOE_ERR_ARG;
  for (int kd = 0; kd < 3; kd++)
    if (!L->kind[kd].row_slot) return MOE_ERR_ARG;
  if (kind < -1 || kind > 2) return MOE_ERR_ARG;
  if (kind == -1 && n_on != 0) return MOE_ERR_ARG;
  const int E = L->n_experts;
  hipStream_t s = static_cast<hipStream_t>(stream);

  if (kind >= 0) {
    const moe_kind_desc_t& K = L->kind[kind];
    const int R = rows_of_kind(L, kind);
    if (n_on < 0 || n_on > K.n_slots) return MOE_ERR_SLOT;
    if (n_on > 0 && (!slots_on || !K.copy_hdr || !K.copy_hdr_host || !L->staging))
      return MOE_ERR_ARG;
    // duplicate slots and two slots on one (expert, row): one flag per slot
    // and one per row of the kind (E*R bytes, reused across calls)
    static thread_local std::vector<uint8_t> seen, rows;
    seen.assign(static_cast<size_t>(K.n_slots), 0);
    rows.assign(static_cast<size_t>(E) * R, 0);
    for (int i = 0; i < n_on; i++) {
      const int sl = slots_on[i];
      if (sl < 0 || sl >= K.n_slots || seen[sl]) return MOE_ERR_SLOT;
      seen[sl] = 1;
      const int e = K.copy_hdr_host[2 * sl];
      const int r = K.copy_hdr_host[2 * sl + 1];
      if (e < 0 || e >= E || r < 0 || r >= R) return MOE_ERR_SLOT;
      uint8_t& f = rows[static_cast<size_t>(e) * R + r];
      if (f) return MOE_ERR_SLOT;
      f = 1;
    }
    if (n_on > 0 &&
        hipMemcpyAsync(L->staging, slots_on, sizeof(int32_t) * n_on, hipMemcpyHostToDevice, s) !=
            hipSuccess)
      return MOE_ERR_HIP;
    const int64_t n = static_cast<int64_t>(E) * R;
    hipLaunchKernelGGL(fill_kernel, dim3(static_cast<unsigned>(cdiv(n, 256))), dim3(256), 0, s,
                       K.row_slot, n, -1);
    if (n_on > 0)
      hipLaunchKernelGGL(scatter_slots_kernel, dim3(static_cast<unsigned>(cdiv(n_on, 256))),
                         dim3(256), 0, s, L->staging, n_on, K.copy_hdr, R, K.row_slot);
  } else {
    for (int kd = 0; kd < 3; kd++) {
      const int64_t n = static_cast<int64_t>(E) * rows_of_kind(L, kd);
      hipLaunchKernelGGL(fill_kernel, dim3(static_cast<unsigned>(cdiv(n, 256))), dim3(256), 0, s,
                         L->kind[kd].row_slot, n, -1);
    }
  }
  if (kind != MOE_KIND_DOWN)
    hipLaunchKernelGGL(order_kernel, dim3(E), dim3(kOrderWaves * kWave), 0, s, L->kind[0].row_slot,
                       static_cast<const int32_t*>(L->kind[1].row_slot), L->d_ff, L->order_gu,
                       L->class_cnt);
  if (kind == MOE_KIND_DOWN || kind == -1)
    hipLaunchKernelGGL(order_kernel, dim3(E), dim3(kOrderWaves * kWave), 0, s, L->kind[2].row_slot,
                       static_cast<const int32_t*>(nullptr), L->d_model, L->order_dn,
                       L->class_cnt + 4 * E);
  return launch_status(s);
}
