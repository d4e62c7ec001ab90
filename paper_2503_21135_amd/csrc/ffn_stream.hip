// ffn.hip -- moe_expert_ffn_mixed: the routed and shared expert FFNs of one
// MoE layer over per-expert mixed-precision packed weights (2/3/4/6/8-bit
// codes, fp16 scale and zero per group of `group` inputs), with the channel
// switch applied row by row.
//
// Sec. IV-A: every expert has its own precision.  Sec. IV-B / V-A: a switched
// row reads its cached 8-bit copy instead of its base codes.  Sec. V-B: the
// packed codes are loaded in wide words, unpacked on chip, dequantized and fed
// to the matrix cores in one fused kernel.
//
// Dequantization, MI355X style.  The codes are turned into bf16 integers
// without any multiply: for b <= 4 a code q is OR-ed into the mantissa of the
// bf16 constant 128.0, giving exactly 128 + q; 8-bit codes go through the
// byte-to-float converter and give q.  The matrix cores then contract these
// exact integers with the bf16 activations in fp32, one quantization group
// at a time, and the group's scale and zero point are applied to the fp32
// partial sum:  sum_c s (q_c - z) x_c = s * (P - (off + z) * X),
// P = sum_c (off + q_c) x_c from the MFMA, X = sum_c x_c over the group.
// The weight operand is therefore exact; the only rounding besides fp32
// accumulation is the bf16 hidden activation h.
//
// Work decomposition (one wave = 64 lanes):
//   - a wave owns 16 rows (neurons for gate/up, output channels for down) of
//     one expert and streams its packed rows through all groups of K (down:
//     one of n_split slices of K);
//   - lane (r16 = lane % 16, kq = lane / 16) loads the group codes
//     [kq*g/4, (kq+1)*g/4) of row r16 -- one 16-byte load at 4 bits -- and
//     the matching activations of token r16 of the current 16-token tile;
//   - v_mfma_f32_16x16x32_bf16 with A = activations (tokens) and
//     B = weights (rows) leaves each lane the results of its own row r16 for
//     tokens 4*kq .. 4*kq+3, so the lane applies its own row's scale/zero.
#include "ffn_common.hpp"

namespace moe {
namespace ffn {

// ------------------------------------------------------------------ streaming kernel
// One workgroup = kWavesOf<NK, VEC> waves on one expert and one source class of
// its rows.  Each wave owns 16 consecutive positions of the expert's row order for
// each of NK weight kinds (NK = 2: the gate and up rows of the same neurons;
// NK = 1: down rows = output channels).  Within a class every kind has one
// source for all rows -- the expert's base codes at bit-width B, or the
// cached 8-bit copies -- so the loads are wave-uniform in shape and the code
// registers are sized for that width (template BG / BU).  The packed codes of
// the next kStages<BG, BU> groups are in flight in registers while the current group
// is dequantized and contracted; the activations of the workgroup's token
// tile (NT*16 rows) are staged in LDS two groups at a time (double-buffered,
// one barrier per two groups), so every wave reads them from LDS.

// Groups of codes in flight per wave: four, or two when a kind streams 8- or
// 6-bit codes (about the same bytes in flight in half the registers).  The activations
// of chunk c+2 are loaded while chunk c is contracted, so that waiting for
// them (vector loads complete in order) never waits for a code load the loop
// does not already need: with two-group chunks that holds for up to four
// groups in flight.
template <int BG, int BU>
constexpr int kStages = (BG >= 8 || BU >= 8 || BG == 6 || BU == 6) ? 2 : 4;

// Metadata a workgroup loads in its prologue, all issued before any is
// waited for (a chain of dependent loads at the start of every workgroup
// costs more than the loads themselves).
struct Pre {
  int64_t code_off[2], sz_off[2];   // per kind of the launch
  int tt, n_tt;                     // token tile of the workgroup, when the tiles are split over workgroups
  int row;                          // class 0: row at lane % 16 of the wave's positions
};

template <int NM, int B>
constexpr int kWords = NM * B / 4;   // code words per lane per group

template <int NM, int BG, int BU>
struct Stage {
  uint32_t cg[(kWords<NM, BG>)];
  uint32_t cu[(kWords<NM, BU>)];   // unused for NK = 1
};

// Source of one kind for a workgroup: resources over the expert's codes and
// {scale, zero} words (or the copies), the per-group stride of the {s, z}
// words and the lane's byte offsets (kOOB for lanes past the rows of the
// class).  The per-group advance goes into the scalar offset of the loads.
struct Src {
  Rsrc code, sz;
  uint32_t sz_gstride;   // bytes between consecutive groups' {s, z} words
  uint32_t coff;         // byte offset of the lane's code share of group 0
  uint32_t soff;         // byte offset of the row's {s, z} word of group 0
};

template <int NM, int B>
__device__ __forceinline__ void load_kind(uint32_t (&cw)[(kWords<NM, B>)], const Src& s, int gi, bool gv) {
  constexpr uint32_t gcb = NM * 32 * B / 8;   // code bytes per row and group
  const uint32_t cadv = gv ? static_cast<uint32_t>(gi) * gcb : 0u;
  bload<kWords<NM, B>>(cw, s.code, gv ? s.coff : kOOB, cadv);
}

// {s, z} words of the four groups [gb, gb+4): lane (r16, kq) loads row r16's
// word of group gb + kq (zero past g1), one load per kind for four groups; each
// group then reads its word from lane r16 + 16*(g - gb).
template <int NK>
__device__ __forceinline__ void load_sz4(uint32_t (&szb)[2], const Src (&src)[2], int gb, int g1, int kq) {
  const bool ok = gb + kq < g1;
#pragma unroll
  for (int kk = 0; kk < NK; kk++) {
    const uint32_t sadv = gb < g1 ? static_cast<uint32_t>(gb) * src[kk].sz_gstride : 0u;
    const uint32_t so = src[kk].soff;
    const uint32_t voff = (ok && so != kOOB) ? so + static_cast<uint32_t>(kq) * src[kk].sz_gstride : kOOB;
    szb[kk] = __builtin_amdgcn_raw_buffer_load_b32(src[kk].sz, voff, sadv, 0);
  }
}

template <int NM, int NK, int BG, int BU>
__device__ __forceinline__ void load_stage(Stage<NM, BG, BU>& st, const Src (&src)[2], int gi, bool gv) {
  load_kind<NM, BG>(st.cg, src[0], gi, gv);
  if constexpr (NK == 2) load_kind<NM, BU>(st.cu, src[1], gi, gv);
}

// Contract one group: A fragments (activations) come from LDS.
//
// All MFMA chains of the group are issued first and their results are read
// only after an explicit wait: a matrix-core result must not be read by a
// VALU instruction before the MFMA has finished writing it, and the code
// around this loop has short control-flow paths on which the compiler's own
// wait-state insertion was observed to fall short (the last accumulator
// element was read stale).  The 3 x s_nop 7 (24 wait states) cover the
// longest 16x16x32 bf16 MFMA latency on gfx950.
template <int NM, int NT, int Bk>
__device__ __forceinline__ void contract_kind(const uint32_t (&cw)[(kWords<NM, Bk>)], uint32_t szw,
                                              const u32x4 (&af)[NT][NM], uint32_t vm, uint32_t vh,
                                              f32x4 (&tmp)[NT], float& sc, float& zz) {
  u32x4 wf[kPlanes<Bk>][NM];
  dequant_b<Bk, NM, kWords<NM, Bk>>(cw, wf, vm, vh);
  sc = fp16_bits_to_f32(szw & 0xFFFFu);
  zz = fp16_bits_to_f32(szw >> 16) + kOffset<Bk>;
#pragma unroll
  for (int nt = 0; nt < NT; nt++) {
    f32x4 t = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int m = 0; m < NM; m++)
#pragma unroll
      for (int pl = 0; pl < kPlanes<Bk>; pl++) t = mfma16(af[nt][m], wf[pl][m], t);
    tmp[nt] = t;
  }
}

template <int NM, int NT, int NK, int BG, int BU>
__device__ __forceinline__ void compute_group(const Stage<NM, BG, BU>& st, const uint32_t (&szw)[2],
                                              const u32x4 (&af)[NT][NM], const f32x4 (&X)[NT],
                                              uint32_t vm, uint32_t vh, f32x4 (&acc)[NK][NT]) {
  f32x4 tmp[NK][NT];
  float sc[NK], zz[NK];
  contract_kind<NM, NT, BG>(st.cg, szw[0], af, vm, vh, tmp[0], sc[0], zz[0]);
  if constexpr (NK == 2) contract_kind<NM, NT, BU>(st.cu, szw[1], af, vm, vh, tmp[1], sc[1], zz[1]);
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 7\n\ts_nop 7\n\ts_nop 7");
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int kk = 0; kk < NK; kk++)
#pragma unroll
    for (int nt = 0; nt < NT; nt++)
#pragma unroll
      for (int i = 0; i < 4; i++)
        acc[kk][nt][i] = __fmaf_rn(sc[kk], __fmaf_rn(-zz[kk], X[nt][i], tmp[kk][nt][i]), acc[kk][nt][i]);
}

// Groups per LDS chunk of activations.  (Four-group chunks halve the
// barriers but double the tile's LDS, which limits the occupancy of the
// down projection; two measured faster.)
constexpr int kChunk = 2;

template <int NM, int NT>
struct XTile {
  static constexpr int g = NM * 32;
  static constexpr int CG = kChunk;
  static constexpr int KC = CG * g;   // K columns per LDS chunk
  static constexpr int TOK = NT * 16;
  static constexpr int LDW = KC + 8;  // row stride in bf16 (16-byte pad)
  uint16_t x[2][TOK][LDW];
  float xs[2][CG][TOK];
};

// fp32 sum of the bf16 values of a group held by g/8 adjacent lanes, 8 each:
// dot products with ones inside the lane, then a tree over the lanes (lane
// pairs, quads, eights, sixteens); every lane gets the sum.  Every workgroup
// forms the sums of the tokens it stages: ~16 VALU instructions per wave and
// group at 32-token tiles, which costs the Mixtral-shaped layer's gate/up launch
// 3 % at 64 tokens, but two launches (5 us each) less than sums made
// beforehand: whole calls 118.2 -> 112.4 us (DeepSeek-shaped, 17 tokens),
// 104.0 -> 99.0 (Mixtral-shaped, 1 token), 257.6 -> 252.0 (64 tokens).
template <int CTRL>
__device__ __forceinline__ float lane_add(float v) {
  return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// acc + sum over the 8 bf16 pairs of a and b
__device__ __forceinline__ float dot8(const u32x4& a, const u32x4& b, float acc) {
#pragma unroll
  for (int c = 0; c < 4; c++) {
    const uint32_t x = a[c], w = b[c];   // a bit cast of a vector element itself takes element 0 in this compiler
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, x), __builtin_bit_cast(bf16x2, w), acc, false);
  }
  return acc;
}

constexpr uint32_t kOnes = 0x3F803F80u;   // two bf16 1.0

template <int g>
__device__ __forceinline__ float group_sum(const u32x4& v) {
  float s = dot8(v, u32x4{kOnes, kOnes, kOnes, kOnes}, 0.f);
  s = lane_add<0xB1>(s);    // quad_perm 1,0,3,2
  s = lane_add<0x4E>(s);    // quad_perm 2,3,0,1
  s = lane_add<0x141>(s);   // row_half_mirror
  if constexpr (g == 128) s = lane_add<0x140>(s);   // row_mirror
  return s;
}

// The rows at order positions [pos0, pos1) of expert e (lanes past pos1
// idle), class cls (bit kk set: kind kk reads the 8-bit copies), token tile
// passes over the expert's segment, K groups [g0, g1) of split sp.
template <int NM, int NT, int NK, int BG, int BU, int WV>
__device__ __forceinline__ void stream_body(const FfnArgs& a, XTile<NM, NT>& tl, const Pre& pre, int e,
                                            int cls, int pos0, int pos1, int R, int sp, int n_split) {
  constexpr int kThreads = 64 * WV;
  constexpr int g = NM * 32;
  constexpr int KC = XTile<NM, NT>::KC;
  constexpr int TOK = XTile<NM, NT>::TOK;
  constexpr int PIECES = TOK * KC / 8;   // 16-byte pieces per chunk
  constexpr int PPT = (PIECES + kThreads - 1) / kThreads;
  static_assert(PIECES % kThreads == 0 || PIECES < kThreads, "chunk must split evenly over the workgroup");
  constexpr int S = kStages<BG, BU>;
  constexpr int CG = XTile<NM, NT>::CG;
  static_assert((S == 2 || S == 4) && CG == 2, "the loop body below handles two two-group chunks");
  static_assert(PPT <= g / 8, "one lane per piece writes a group sum");
  const int tid = threadIdx.x;
  const int wv = tid >> 6;
  const int lane = tid & 63;
  const int r16 = lane & 15;
  const int kq = lane >> 4;
  const int seg0 = uni(a.offsets[e]);
  const int seg1 = uni(a.offsets[e + 1]);
  const bool routed = e < a.E;
  const bool down = NK == 1;
  const int K = down ? (routed ? a.f : a.fs) : a.d;
  const int G = K / g;
  const int g0 = sp * G / n_split;
  const int g1 = (sp + 1) * G / n_split;
  const int be = BG == BU ? BG : (cls == 1 ? BU : BG);   // the base width of the expert
  const int kind0 = down ? 2 : 0;
  const int32_t* order = down ? a.order_dn : a.order_gu;

  const int pos = pos0 + wv * 16 + r16;
  const bool live = pos < pos1;
  // positions past the class (pos >= pos1) are not read: for the last expert's
  // last class they would lie past the end of the order table
  int prow = pre.row;
  if (cls != 0) prow = live ? order[static_cast<int64_t>(e) * R + pos] : 0;
  const int row_id = live ? prow : 0;
  // a wave whose rows all lie past the class (the last workgroup of an
  // expert whose rows do not fill it) still stages activations and meets the
  // barriers, but contracts nothing
  const bool wave_live = uni(pos0 + wv * 16) < pos1;
  Src src[2];
#pragma unroll
  for (int kk = 0; kk < NK; kk++) {
    // scalar selects first, one resource each: a resource chosen by a branch
    // would be merged in vector registers and force a loop per load
    const KindDev& kd = a.kd[kind0 + kk];
    const bool copy = (cls >> kk) & 1;
    const uint32_t row_bytes = 4u * static_cast<uint32_t>(code_row_words(K, be));
    const uint32_t words = static_cast<uint32_t>(g) * be / 128;   // per lane per group
    const void* cptr = copy ? static_cast<const void*>(kd.copy_codes)
                            : static_cast<const void*>(kd.codes + uni(pre.code_off[kk]));
    const void* sptr = copy ? static_cast<const void*>(kd.copy_sz)
                            : static_cast<const void*>(kd.sz + uni(pre.sz_off[kk]));
    const uint32_t cbytes = copy ? a.copy_bytes[kind0 + kk] : static_cast<uint32_t>(R) * row_bytes;
    const uint32_t sbytes = copy ? a.copy_sz_bytes[kind0 + kk] : static_cast<uint32_t>(R) * G * 4u;
    Src& s = src[kk];
    s.code = make_rsrc(cptr, cbytes);
    s.sz = make_rsrc(sptr, sbytes);
    s.sz_gstride = copy ? 4u : static_cast<uint32_t>(R) * 4u;
    const int slot = (copy && live) ? kd.row_slot[static_cast<int64_t>(e) * R + row_id] : -1;
    const uint32_t c_base = live ? row_id * row_bytes + kq * words * 4u : kOOB;
    const uint32_t s_base = live ? row_id * 4u : kOOB;
    const uint32_t c_copy =
        slot >= 0 ? static_cast<uint32_t>(slot) * 4u * static_cast<uint32_t>(code_row_words(K, 8)) + kq * (g / 4) : kOOB;
    const uint32_t s_copy = slot >= 0 ? static_cast<uint32_t>(slot) * G * 4u : kOOB;
    s.coff = copy ? c_copy : c_base;
    s.soff = copy ? s_copy : s_base;
  }
  const Rsrc xr = make_rsrc(down ? a.h : a.x, down ? a.h_bytes : a.x_bytes);

  // token tiles pre.tt, pre.tt + n_tt, ... of the segment (all of them
  // when the launch has one workgroup set per row block)
  for (int t0 = seg0 + pre.tt * TOK; t0 < seg1; t0 += pre.n_tt * TOK) {
    // piece q = tid + kThreads*i of a chunk: token row q / (KC/8), column (q % (KC/8))*8
    uint32_t arow[PPT];   // byte offset of the token's row, kOOB when absent
#pragma unroll
    for (int i = 0; i < PPT; i++) {
      const int p = t0 + (tid + kThreads * i) / (KC / 8);
      arow[i] = p < seg1 && tid + kThreads * i < PIECES ? static_cast<uint32_t>(2 * (down ? h_row(a, p)
                                                          : static_cast<int64_t>(a.perm[p]) * K))
                         : kOOB;
    }
    const int acol = (tid % (KC / 8)) * 8;   // same column for every piece of a thread
#pragma unroll
    for (int i = 0; i < PPT; i++)
      if (arow[i] != kOOB) arow[i] += 2u * acol;
    // chunk [gc, gc+CG): the chunk's first column goes into the scalar offset
    auto stage_x = [&](u32x4 (&v)[PPT], int gc) {
      const uint32_t xadv = gc < g1 ? 2u * static_cast<uint32_t>(gc * g) : 0u;
      const bool in_k = gc + acol / g < g1;   // the chunk's later groups may not exist
#pragma unroll
      for (int i = 0; i < PPT; i++) v[i] = bload4(xr, in_k ? arow[i] : kOOB, xadv);
    };
    // Writes the chunk to LDS, and each token's group sums: the g/8 adjacent
    // lanes that hold one group of a token add their pieces, and lane i of
    // them writes the sum of piece i.
    const int ql = tid % (g / 8);
    float* const xs_dst = &tl.xs[0][acol / g][(tid + kThreads * min(ql, PPT - 1)) / (KC / 8)];
    const bool xs_own = ql < PPT && (PIECES >= kThreads || tid < PIECES);
    auto write_x = [&](const u32x4 (&v)[PPT], int buf) {
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < PPT; i++) {
        if (PIECES >= kThreads || tid < PIECES)
          *reinterpret_cast<u32x4*>(&tl.x[buf][(tid + kThreads * i) / (KC / 8)][acol]) = v[i];
        const float s = group_sum<g>(v[i]);
        sum = i == 0 || ql == i ? s : sum;
      }
      if (xs_own) xs_dst[buf * (CG * TOK)] = sum;
    };

    f32x4 acc[NK][NT];
#pragma unroll
    for (int kk = 0; kk < NK; kk++)
#pragma unroll
      for (int nt = 0; nt < NT; nt++) acc[kk][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // dequantization constants, kept in vector registers (see dequant_b)
    uint32_t vm = kMagic, vh = kHighMagic<BG, BU>;
    asm volatile("" : "+v"(vm), "+v"(vh));
    Stage<NM, BG, BU> st[S];
#pragma unroll
    for (int s = 0; s < S; s++) load_stage<NM, NK, BG, BU>(st[s], src, g0 + s, g0 + s < g1);
    u32x4 vx[CG == 2 ? 2 : 1][PPT];   // activations of the next chunk(s)
    uint32_t szc[2], szn[2];   // {s, z} words of this and the next four groups
    load_sz4<NK>(szc, src, g0, g1, kq);
    stage_x(vx[0], g0);
    write_x(vx[0], 0);
    if constexpr (CG == 2) stage_x(vx[1], g0 + 2);
    __syncthreads();
    auto group = [&](Stage<NM, BG, BU>& s, int buf, int gg, int gi, int i4) {
      if (gi < g1 && wave_live) {   // wave-uniform; the loads below are unconditional
        uint32_t szw[2];
#pragma unroll
        for (int kk = 0; kk < NK; kk++)
          szw[kk] = static_cast<uint32_t>(__shfl(static_cast<int>(szc[kk]), r16 + 16 * i4));
        u32x4 af[NT][NM];
        f32x4 X[NT];
#pragma unroll
        for (int nt = 0; nt < NT; nt++) {
#pragma unroll
          for (int m = 0; m < NM; m++)
            af[nt][m] = *reinterpret_cast<const u32x4*>(&tl.x[buf][nt * 16 + r16][gg * g + kq * (g / 4) + 8 * m]);
          X[nt] = *reinterpret_cast<const f32x4*>(&tl.xs[buf][gg][nt * 16 + 4 * kq]);
        }
        compute_group<NM, NT, NK, BG, BU>(s, szw, af, X, vm, vh, acc);
      }
      load_stage<NM, NK, BG, BU>(s, src, gi + S, gi + S < g1);
    };
    for (int gc = g0; gc < g1; gc += 4) {
#pragma unroll
      for (int c = 0; c < 2; c++) {   // chunk c of the iteration sits in LDS buffer c
        // vx[c] held chunk gc+2c (written to LDS already); reuse it for gc+2c+4
        stage_x(vx[c], gc + 2 * c + 4);
        group(st[(2 * c) % S], c, 0, gc + 2 * c, 2 * c);
        if (c == 0) load_sz4<NK>(szn, src, gc + 4, g1, kq);
        group(st[(2 * c + 1) % S], c, 1, gc + 2 * c + 1, 2 * c + 1);
        write_x(vx[c ^ 1], c ^ 1);   // chunk gc+2c+2, loaded one chunk ago
        __syncthreads();
      }
#pragma unroll
      for (int kk = 0; kk < NK; kk++) szc[kk] = szn[kk];
    }

    if constexpr (NK == 2) {
      // SiLU-GLU epilogue: h = bf16(silu(g) * u)
#pragma unroll
      for (int nt = 0; nt < NT; nt++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const int p = t0 + nt * 16 + 4 * kq + i;
          if (live && p < seg1) {
            const float hv = silu_mul(acc[0][nt][i], acc[1][nt][i]);
            a.h[h_row(a, p) + row_id] = static_cast<uint16_t>(bf16_rne(hv));
          }
        }
    } else {
      float* out = a.o + static_cast<int64_t>(sp) * a.split_stride;
#pragma unroll
      for (int nt = 0; nt < NT; nt++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const int p = t0 + nt * 16 + 4 * kq + i;
          if (live && p < seg1) out[static_cast<int64_t>(p) * R + row_id] = acc[0][nt][i];
        }
    }
  }
}


// ------------------------------------------------------------------ one or two tokens
// For batches of one or two tokens (kVecTok) the matrix tile would be mostly
// padding, and the streaming body is bound by latency and by the L1: its lanes
// hold 16 rows, so a load instruction touches 16 rows' cache lines 16 bytes at
// a time, and the activation chunks tie four waves to a barrier.  Here a wave
// takes its 16 rows one after another, its lanes side by side along K: four
// lanes per group, 16 groups of a row per load (1 KB in a row at 4 bits), the
// activations of the lane's columns in registers, no LDS and no barrier.  The
// codes become the same exact bf16 integers, which v_dot2_f32_bf16 contracts
// in fp32 with the lane's activations; the lane applies its group's scale and
// zero point to its own partial sum, and the lanes' sums are added at the end.
// Eight rows' codes are in flight.
// Whole calls against 16-token tiles (repeated calls, weights partly in the
// Infinity Cache): Mixtral-shaped 97.3 -> 79.7 us at 1 token and 108.9 -> 104.7 at
// 2, DeepSeek-shaped 60.3 -> 50.0 and 63.1 -> 57.8, Qwen-shaped 66.2 -> 54.8 and
// 72.4 -> 62.4.  With more tokens the launch has waves enough and the matrix tile's
// fewer instructions per weight win: at 3 tokens 148.1 -> 140.6, 63.9 -> 66.5 and
// 73.1 -> 77.8, at 4 148.1 -> 169.6, 69.6 -> 73.4 and 75.5 -> 83.0; chosen per
// expert by its token count it lost 2 to 13 % from 3 to 20 tokens on the
// DeepSeek-shaped layer and up to 6 % from 6 on the Mixtral-shaped one.

// Sums of N values (a power of two, at most 64) over the wave: at each offset a
// lane keeps half of its values and hands the other half over; value v ends in
// the lanes l with l / (64 / N) == v.
template <int N, int OFF, int NV>
__device__ __forceinline__ void wave_scatter_sum(float (&v)[NV], int lane) {
  if constexpr (OFF >= 1) {
    constexpr int H = N > 1 ? N / 2 : 1;
    if constexpr (N > 1) {
      const bool hi = (lane & OFF) != 0;
#pragma unroll
      for (int i = 0; i < H; i++) {
        const float send = hi ? v[i] : v[i + H];
        const float keep = hi ? v[i + H] : v[i];
        v[i] = keep + __shfl_xor(send, OFF, kWave);
      }
    } else {
      v[0] = v[0] + __shfl_xor(v[0], OFF, kWave);
    }
    wave_scatter_sum<H, OFF / 2, NV>(v, lane);
  }
}

// The rows at order positions [pos0, pos1) of expert e on its base codes,
// TT rows of its segment from seg0 on, K groups [g0, g1) of split sp.
template <int NM, int NK, int B, int TT>
__device__ __forceinline__ void vec_body(const FfnArgs& a, const Pre& pre, int e, int pos0, int pos1, int R, int sp,
                                         int n_split, int seg0) {
  constexpr int g = NM * 32;
  constexpr int NW = kWords<NM, B>;
  constexpr int RB = NK * TT == 4 ? 8 : 16;   // rows whose sums a lane holds at once
  constexpr int D = 8 / NK;                   // rows in flight
  constexpr int N = RB * TT;
  constexpr uint32_t gcb = NM * 32 * B / 8;   // code bytes per row and group
  const int lane = threadIdx.x & 63;
  const int p0 = pos0 + 16 * uni(static_cast<int>(threadIdx.x >> 6));
  if (p0 >= pos1) return;
  const int n_rows = min(16, pos1 - p0);
  const bool routed = e < a.E;
  const bool down = NK == 1;
  const int K = down ? (routed ? a.f : a.fs) : a.d;
  const int G = K / g;
  const int g0 = sp * G / n_split;
  const int g1 = (sp + 1) * G / n_split;
  const int kind0 = down ? 2 : 0;
  // lane r holds row r (past the class: its last row, computed and not stored)
  const int row = __shfl(pre.row, min(lane & 15, n_rows - 1));
  const uint32_t row_bytes = 4u * static_cast<uint32_t>(code_row_words(K, B));
  Rsrc code[NK], sz[NK];
#pragma unroll
  for (int kk = 0; kk < NK; kk++) {
    const KindDev& kd = a.kd[kind0 + kk];
    code[kk] = make_rsrc(kd.codes + uni(pre.code_off[kk]), static_cast<uint32_t>(R) * row_bytes);
    sz[kk] = make_rsrc(kd.sz + uni(pre.sz_off[kk]), static_cast<uint32_t>(R) * G * 4u);
  }
  const Rsrc xr = make_rsrc(down ? a.h : a.x, down ? a.h_bytes : a.x_bytes);
  uint32_t xrow[TT];   // byte offset of the token's row
#pragma unroll
  for (int t = 0; t < TT; t++) {
    const int p = seg0 + t;
    xrow[t] = uni(static_cast<uint32_t>(2 * (down ? h_row(a, p) : static_cast<int64_t>(a.perm[p]) * K)));
  }
  uint32_t vm = kMagic, vh = kHighMagic<B, B>;
  asm volatile("" : "+v"(vm), "+v"(vh));

  for (int rb = 0; rb < n_rows; rb += RB) {
    float acc[NK][N];
#pragma unroll
    for (int kk = 0; kk < NK; kk++)
#pragma unroll
      for (int i = 0; i < N; i++) acc[kk][i] = 0.f;
    for (int gc = g0; gc < g1; gc += 16) {
      const int gi = gc + (lane >> 2);
      const bool ok = gi < g1;   // lanes past the slice read zeros everywhere
      const uint32_t xo = ok ? static_cast<uint32_t>(2 * (gi * g + (lane & 3) * (g / 4))) : kOOB;
      const uint32_t co = ok ? static_cast<uint32_t>(gi) * gcb + (lane & 3) * (gcb / 4) : kOOB;
      const uint32_t so = ok ? static_cast<uint32_t>(gi) * static_cast<uint32_t>(R) * 4u : kOOB;
      uint32_t cw[D][NK][NW], sw[D][NK];
      auto load = [&](int r) {
        const uint32_t rid = static_cast<uint32_t>(__builtin_amdgcn_readlane(row, rb + r));
#pragma unroll
        for (int kk = 0; kk < NK; kk++) {
          bload<NW>(cw[r % D][kk], code[kk], co, rid * row_bytes);
          sw[r % D][kk] = __builtin_amdgcn_raw_buffer_load_b32(sz[kk], so, rid * 4u, 0);
        }
      };
      u32x4 x[TT][NM];
      float X[TT];
#pragma unroll
      for (int t = 0; t < TT; t++)
#pragma unroll
        for (int m = 0; m < NM; m++) x[t][m] = bload4(xr, ok ? xo + 16u * m : kOOB, xrow[t]);
#pragma unroll
      for (int r = 0; r < D; r++) load(r);
#pragma unroll
      for (int t = 0; t < TT; t++) {
        X[t] = 0.f;
#pragma unroll
        for (int m = 0; m < NM; m++) X[t] = dot8(x[t][m], u32x4{kOnes, kOnes, kOnes, kOnes}, X[t]);
      }
#pragma unroll
      for (int r = 0; r < RB; r++) {
#pragma unroll
        for (int kk = 0; kk < NK; kk++) {
          u32x4 wf[kPlanes<B>][NM];
          dequant_b<B, NM, NW>(cw[r % D][kk], wf, vm, vh);
          const uint32_t w = sw[r % D][kk];
          const float sc = fp16_bits_to_f32(w & 0xFFFFu);
          const float zz = fp16_bits_to_f32(w >> 16) + kOffset<B>;
#pragma unroll
          for (int t = 0; t < TT; t++) {
            float s = 0.f;   // a chain of dependent dot products per operand, then their sum
#pragma unroll
            for (int m = 0; m < NM; m++) {
              float sm = 0.f;
#pragma unroll
              for (int pl = 0; pl < kPlanes<B>; pl++) sm = dot8(x[t][m], wf[pl][m], sm);
              s = m == 0 ? sm : s + sm;
            }
            acc[kk][r * TT + t] = __fmaf_rn(sc, __fmaf_rn(-zz, X[t], s), acc[kk][r * TT + t]);
          }
        }
        if (r + D < RB) load(r + D);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int kk = 0; kk < NK; kk++) wave_scatter_sum<N, kWave / 2, N>(acc[kk], lane);
    const int v = lane / (kWave / N);
    const int r = rb + v / TT, t = v % TT;
    const int rid = __shfl(row, r & 15);
    if (lane % (kWave / N) == 0 && r < n_rows) {
      const int p = seg0 + t;
      if constexpr (down)
        a.o[static_cast<int64_t>(sp) * a.split_stride + static_cast<int64_t>(p) * R + rid] = acc[0][0];
      else
        a.h[h_row(a, p) + rid] = static_cast<uint16_t>(bf16_rne(silu_mul(acc[0][0], acc[NK - 1][0])));
    }
  }
}

// The expert's segment two rows at a time.  Routing gives an expert at most
// kVecTok rows of a batch this small, but a caller's own offsets may give it up
// to T*k (a token that names an expert more than once).
template <int NM, int NK, int B>
__device__ __forceinline__ void vec_dispatch(const FfnArgs& a, const Pre& pre, int e, int pos0, int pos1, int R,
                                             int sp, int n_split, int seg0, int seg1) {
#pragma nounroll
  for (; seg1 - seg0 > 1; seg0 += 2) vec_body<NM, NK, B, 2>(a, pre, e, pos0, pos1, R, sp, n_split, seg0);
  if (seg0 < seg1) vec_body<NM, NK, B, 1>(a, pre, e, pos0, pos1, R, sp, n_split, seg0);
}


// Class 0: both kinds on the expert's base codes (in the VEC kernel vec_body's);
// the switched classes have one or both kinds on the 8-bit copies.
template <int NM, int NT, int NK, int B, int WV, bool VEC>
__device__ __forceinline__ void dispatch_class(const FfnArgs& a, XTile<NM, NT>& tl, const Pre& pre, int e,
                                               int cls, int pos0, int pos1, int R, int sp, int n_split) {
  if constexpr (NK == 1) {
    if (!VEC && cls == 0) stream_body<NM, NT, 1, B, B, WV>(a, tl, pre, e, 0, pos0, pos1, R, sp, n_split);
    else stream_body<NM, NT, 1, 8, 8, WV>(a, tl, pre, e, 1, pos0, pos1, R, sp, n_split);
  } else {
    if (!VEC && cls == 0) stream_body<NM, NT, 2, B, B, WV>(a, tl, pre, e, 0, pos0, pos1, R, sp, n_split);
    else if (cls == 1) stream_body<NM, NT, 2, 8, B, WV>(a, tl, pre, e, 1, pos0, pos1, R, sp, n_split);
    else if (cls == 2) stream_body<NM, NT, 2, B, 8, WV>(a, tl, pre, e, 2, pos0, pos1, R, sp, n_split);
    else stream_body<NM, NT, 2, 8, 8, WV>(a, tl, pre, e, 3, pos0, pos1, R, sp, n_split);
  }
}

// Local index l of a workgroup inside a run of nblk row blocks with m
// variants each (token-tile sets x K slices) -> (block, variant).  Blocks
// go in chunks of 8 with the variant outside the block inside a chunk, so
// the variants of one block are 8 workgroups apart: the hardware places
// workgroup b on XCD b % 8, so they run on one XCD and share its L2 (the
// block's codes are read from HBM once).
__device__ __forceinline__ void block_variant(int l, int nblk, int m, int& blk, int& v) {
  const int c = l / (8 * m);
  const int r = l - c * 8 * m;
  const int nb = min(8, nblk - 8 * c);
  v = r / nb;
  blk = 8 * c + (r - v * nb);
}

// One launch serves every streamed expert of a stage: the switched-class
// workgroups of the routed experts first (n_sw per expert, an upper bound on
// what its copies can need; those past its actual class sizes exit at once),
// then the class-0 workgroups of the entries of the map (shared experts,
// then routed experts widest first), as many row blocks per entry of a kind.
template <int NM, int NT, int NK, bool VEC>
__global__ void __launch_bounds__((64 * kWavesOf<NK, VEC>)) __attribute__((amdgpu_waves_per_eu(2)))
ffn_stream_kernel(FfnArgs a, WgMap map) {
  __shared__ __attribute__((aligned(16))) XTile<NM, NT> tl;
  constexpr int WV = kWavesOf<NK, VEC>;
  constexpr int rows1 = WV * 16;   // rows of the workgroup
  const int bid = blockIdx.x;
  const int n_swg = map.n_r * map.n_sw * map.m_r;
  int e, blk, v, B;
  const bool sw = bid < n_swg;
  if (sw) {
    const int per = map.n_sw * map.m_r;
    e = bid / per;
    block_variant(bid - e * per, map.n_sw, map.m_r, blk, v);
    B = map.bits[e / 4] >> (8 * (e % 4)) & 0xFFu;
  } else {
    const int per_s = map.blk_s * map.m_s, per_r = map.blk_r * map.m_r;
    int w = bid - n_swg;
    const bool shared = w < map.n_s * per_s;
    if (!shared) w -= map.n_s * per_s;
    const int i = w / (shared ? per_s : per_r);
    block_variant(w - i * (shared ? per_s : per_r), shared ? map.blk_s : map.blk_r, shared ? map.m_s : map.m_r, blk,
                  v);
    const int ent = map.ent[shared ? i : map.n_s + i];
    e = ent & 0xFFFF;
    B = ent >> 16;
  }
  const bool routed = e < a.E;
  const int n_tt = routed ? map.tt_r : map.tt_s;
  const int tt = v % n_tt, sp = v / n_tt;
  const int R = NK == 1 ? a.d : (routed ? a.f : a.fs);
  const int kind0 = NK == 1 ? 2 : 0;
  // issue every metadata load of the workgroup before waiting for any of them
  const int32_t* ccp = a.class_cnt + (NK == 1 ? 4 * a.E : 0) + 4 * (routed ? e : 0);
  const int o0 = a.offsets[e], o1 = a.offsets[e + 1];
  int cnt[4];
#pragma unroll
  for (int c = 0; c < 4; c++) cnt[c] = ccp[c];
  Pre pre;
  pre.tt = tt;
  pre.n_tt = n_tt;
#pragma unroll
  for (int kk = 0; kk < NK; kk++) {
    pre.code_off[kk] = a.kd[kind0 + kk].code_off[e];
    pre.sz_off[kk] = a.kd[kind0 + kk].sz_off[e];
  }
  {  // class 0 starts at position 0: the wave's rows do not wait for the class sizes
    const int pos = min(blk * rows1 + 16 * static_cast<int>(threadIdx.x >> 6) + static_cast<int>(threadIdx.x & 15), R - 1);
    pre.row = pos;
    if (routed && !sw) pre.row = (NK == 1 ? a.order_dn : a.order_gu)[static_cast<int64_t>(e) * R + pos];
  }
  if (uni(o1) <= uni(o0)) return;
  int cls = 0, start = 0, count = R;
  if (routed) {
#pragma unroll
    for (int c = 0; c < 4; c++) cnt[c] = uni(cnt[c]);
    count = cnt[0];
    if (sw) {   // find the switched class of this workgroup
      start = cnt[0];
      cls = 4;
      for (int c = 1; c < (NK == 1 ? 2 : 4); c++) {
        const int nwg = (cnt[c] + rows1 - 1) / rows1;
        if (blk < nwg) {
          cls = c;
          break;
        }
        blk -= nwg;
        start += cnt[c];
      }
      if (cls == 4) return;
      count = cnt[cls];
    }
  }
  const int pos0 = start + blk * rows1;
  if (blk * rows1 >= count) return;
  const int pos1 = min(pos0 + rows1, start + count);
  const int n_split = map.n_split;
  if constexpr (VEC) {
    if (cls == 0) {
      const int seg0 = uni(o0), seg1 = uni(o1);
      if (B == 8) vec_dispatch<NM, NK, 8>(a, pre, e, pos0, pos1, R, sp, n_split, seg0, seg1);
      else if (NM == 2 && B == 16) {
        if constexpr (NM == 2) vec_dispatch<NM, NK, 16>(a, pre, e, pos0, pos1, R, sp, n_split, seg0, seg1);
      } else if (B == 4) vec_dispatch<NM, NK, 4>(a, pre, e, pos0, pos1, R, sp, n_split, seg0, seg1);
      else if (B == 2) vec_dispatch<NM, NK, 2>(a, pre, e, pos0, pos1, R, sp, n_split, seg0, seg1);
      else if constexpr (NM == 4) {
        if (B == 6) vec_dispatch<NM, NK, 6>(a, pre, e, pos0, pos1, R, sp, n_split, seg0, seg1);
        else vec_dispatch<NM, NK, 3>(a, pre, e, pos0, pos1, R, sp, n_split, seg0, seg1);
      }
      return;
    }
  }
  if constexpr (NT == 2) {
    // an expert with at most 16 tokens needs one 16-token tile: half the
    // contraction and epilogue work of the 32-token tile (same LDS)
    if (uni(o1) - uni(o0) <= 16) {
      auto& t1 = *reinterpret_cast<XTile<NM, 1>*>(&tl);
      if (B == 8) dispatch_class<NM, 1, NK, 8, WV, VEC>(a, t1, pre, e, cls, pos0, pos1, R, sp, n_split);
      else if (NM == 2 && B == 16) {   // unquantized experts need group 64
        if constexpr (NM == 2) dispatch_class<NM, 1, NK, 16, WV, VEC>(a, t1, pre, e, cls, pos0, pos1, R, sp, n_split);
      } else if (B == 4) dispatch_class<NM, 1, NK, 4, WV, VEC>(a, t1, pre, e, cls, pos0, pos1, R, sp, n_split);
      else if (B == 2) dispatch_class<NM, 1, NK, 2, WV, VEC>(a, t1, pre, e, cls, pos0, pos1, R, sp, n_split);
      else if constexpr (NM == 4) {
        if (B == 6) dispatch_class<NM, 1, NK, 6, WV, VEC>(a, t1, pre, e, cls, pos0, pos1, R, sp, n_split);
        else dispatch_class<NM, 1, NK, 3, WV, VEC>(a, t1, pre, e, cls, pos0, pos1, R, sp, n_split);
      }
      return;
    }
  }
  if (B == 8) dispatch_class<NM, NT, NK, 8, WV, VEC>(a, tl, pre, e, cls, pos0, pos1, R, sp, n_split);
  else if (NM == 2 && B == 16) {   // unquantized experts need group 64
    if constexpr (NM == 2) dispatch_class<NM, NT, NK, 16, WV, VEC>(a, tl, pre, e, cls, pos0, pos1, R, sp, n_split);
  } else if (B == 4) dispatch_class<NM, NT, NK, 4, WV, VEC>(a, tl, pre, e, cls, pos0, pos1, R, sp, n_split);
  else if (B == 2) dispatch_class<NM, NT, NK, 2, WV, VEC>(a, tl, pre, e, cls, pos0, pos1, R, sp, n_split);
  else if constexpr (NM == 4) {
    if (B == 6) dispatch_class<NM, NT, NK, 6, WV, VEC>(a, tl, pre, e, cls, pos0, pos1, R, sp, n_split);
    else dispatch_class<NM, NT, NK, 3, WV, VEC>(a, tl, pre, e, cls, pos0, pos1, R, sp, n_split);
  }
}

// Instantiations: every group size by default; a build may compile this file
// once per group size (MOE_FFN_NM = 2 or 4, that is 64 or 128) to spread the
// work over several compiler processes.
#if !defined(MOE_FFN_NM) || MOE_FFN_NM == 2
template __global__ void ffn_stream_kernel<2, 1, 1, false>(FfnArgs, WgMap);
template __global__ void ffn_stream_kernel<2, 1, 1, true>(FfnArgs, WgMap);
template __global__ void ffn_stream_kernel<2, 1, 2, false>(FfnArgs, WgMap);
template __global__ void ffn_stream_kernel<2, 1, 2, true>(FfnArgs, WgMap);
template __global__ void ffn_stream_kernel<2, 2, 1, false>(FfnArgs, WgMap);
template __global__ void ffn_stream_kernel<2, 2, 2, false>(FfnArgs, WgMap);
#endif
#if !defined(MOE_FFN_NM) || MOE_FFN_NM == 4
template __global__ void ffn_stream_kernel<4, 1, 1, false>(FfnArgs, WgMap);
template __global__ void ffn_stream_kernel<4, 1, 1, true>(FfnArgs, WgMap);
template __global__ void ffn_stream_kernel<4, 1, 2, false>(FfnArgs, WgMap);
template __global__ void ffn_stream_kernel<4, 1, 2, true>(FfnArgs, WgMap);
template __global__ void ffn_stream_kernel<4, 2, 1, false>(FfnArgs, WgMap);
template __global__ void ffn_stream_kernel<4, 2, 2, false>(FfnArgs, WgMap);
#endif

}  // namespace ffn
}  // namespace moe
