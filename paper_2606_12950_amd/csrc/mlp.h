// Device code shared by the bfloat16 predictor kernels: MFMA operand layouts, the epilogues that turn
// a row's outputs into a length and KV bytes, and direct global->LDS loads.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace maestro {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Output row (neuron or bin) of a 32x32 MFMA result held in accumulator register v by
// lane-half h (lanes 0-31: h = 0, lanes 32-63: h = 1); the column is the lane's row r.
__device__ __forceinline__ int acc_row(int v, int h) { return (v >> 2) * 8 + h * 4 + (v & 3); }

// 16 consecutive floats of a 32-wide slice as seen by accumulator registers of lane-half h:
// out[v] = src[acc_row(v, h)].
__device__ __forceinline__ void load_acc_layout(const float* __restrict__ src, int h, float (&out)[16]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float4 f = *reinterpret_cast<const float4*>(src + q * 8 + h * 4);
    out[q * 4 + 0] = f.x; out[q * 4 + 1] = f.y; out[q * 4 + 2] = f.z; out[q * 4 + 3] = f.w;
  }
}

// alpha(M) of a stage's model, as float64; a model id outside [0, n_models) gives NaN, so that
// stage's KV demand is NaN and no node admits it.
__device__ __forceinline__ double alpha_of(const float* __restrict__ alpha, int32_t model, int32_t n_models) {
  return (uint32_t)model < (uint32_t)n_models ? (double)alpha[model] : (double)NAN;
}

// Softmax over the B = 32*BT logits of each row, expected length, Eq. 3 KV bytes.
// Lanes r and r + 32 hold complementary halves of row r's logits.
template <int BT>
__device__ __forceinline__ void length_epilogue(const f32x16 (&logit)[BT], const float* __restrict__ b_last,
                                                const float* __restrict__ centre, int h, int64_t row, int64_t n,
                                                int32_t prompt, int32_t model, const float* __restrict__ alpha,
                                                int32_t n_models, float* __restrict__ pred_len,
                                                double* __restrict__ kv_bytes) {
  float z[BT][16], c[BT][16];
  float mx = -INFINITY;
#pragma unroll
  for (int bt = 0; bt < BT; ++bt) {
    float bias[16];
    load_acc_layout(b_last + bt * 32, h, bias);
    load_acc_layout(centre + bt * 32, h, c[bt]);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      z[bt][v] = logit[bt][v] + bias[v];
      mx = fmaxf(mx, z[bt][v]);
    }
  }
  mx = fmaxf(mx, __shfl_xor(mx, 32));
  // e^(z - mx) = 2^((z - mx) log2(e)) with the hardware 2^x; the difference is taken first
  // (exact when z is near mx), so very large logits lose no accuracy to a rounded mx log2(e).
  // The weighted sum of centres accumulates with fused multiply-adds.
  constexpr float kLog2e = 1.4426950408889634f;
  float se = 0.0f, sc = 0.0f;
#pragma unroll
  for (int bt = 0; bt < BT; ++bt) {
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float e = __builtin_amdgcn_exp2f(__fmul_rn(__fsub_rn(z[bt][v], mx), kLog2e));
      se += e;
      sc = fmaf(e, c[bt][v], sc);
    }
  }
  se += __shfl_xor(se, 32);
  sc += __shfl_xor(sc, 32);
  if (h == 0 && row < n) {
    const float pred = sc / se;
    pred_len[row] = pred;
    kv_bytes[row] = ((double)prompt + (double)pred) * alpha_of(alpha, model, n_models);
  }
}

// Per-stage inputs and tables of the two-phase predictor (unused by the bins predictor).
struct TwoPhaseArgs {
  const int32_t* role_id;
  const int32_t* tool_avail;
  const int32_t* role_head;
  const float* tool_coef;
  const float* iso_x;
  const float* iso_y;
  int32_t n_roles;
  int32_t n_knots;
  float max_len;
  float* p_tool;

  TwoPhaseArgs from(int64_t row) const {   // the same for the rows from `row` on
    TwoPhaseArgs t = *this;
    if (t.role_id) t.role_id += row;
    if (t.tool_avail) t.tool_avail += row;
    if (t.p_tool) t.p_tool += row;
    return t;
  }
};

// The B = 32*BT outputs of each row read as heads (Sec. III-B): output 0 the tool-intent
// logit, output g the log(1 + L) regressor of the row's head g (role_head of its role, head 1
// when the role has none). p_tool = iso(sigmoid(z_0)) (Eq. 1 calibrated; 0 without tools),
// L = min(expm1(max(z_g + coef_g p_tool, 0)), max_len), then Eq. 3.
__device__ __forceinline__ int head_of_role(int32_t role, const int32_t* __restrict__ head_of, int32_t n_roles,
                                            int n_out) {
  int g = (role >= 0 && role < n_roles) ? head_of[role] : 1;
  return (g < 1 || g >= n_out) ? 1 : g;
}

// Output g of a row, summed over its two lane-halves: lane-half h holds the outputs
// 32 bt + acc_row(v, h), so exactly one half holds output g, as register v = 4 (t / 8) + t % 4
// of tile bt = g / 32 (t = g % 32) when (t / 4) % 2 == h. A five-level selection tree over the
// register index picks it; the other half contributes 0.
template <int BT>
__device__ __forceinline__ float head_output(const f32x16 (&z)[BT], int g, int h) {
  static_assert(BT == 2, "a 32-entry selection tree");
  const int t = g & 31;
  const int idx = (g >> 5) * 16 + (t >> 3) * 4 + (t & 3);
  float val[32];
#pragma unroll
  for (int bt = 0; bt < BT; ++bt)
#pragma unroll
    for (int v = 0; v < 16; ++v) val[16 * bt + v] = z[bt][v];
#pragma unroll
  for (int lvl = 0; lvl < 5; ++lvl) {
    const bool bit = (idx >> lvl) & 1;
#pragma unroll
    for (int j = 0; j < (16 >> lvl); ++j) val[j] = bit ? val[2 * j + 1] : val[2 * j];
  }
  const float mine = (((t >> 2) & 1) == h) ? val[0] : 0.0f;
  return mine + __shfl_xor(mine, 32);
}

// The rest of one row from its tool-intent output z0 and head output zg (biases not yet added).
__device__ __forceinline__ void two_phase_row(float z0, float zg, int g, const float* __restrict__ b_last,
                                              const float* __restrict__ coef, const float* __restrict__ kx,
                                              const float* __restrict__ ky, const TwoPhaseArgs& tp, int64_t row,
                                              int32_t prompt, int32_t model, int32_t tools,
                                              const float* __restrict__ alpha, int32_t n_models,
                                              float* __restrict__ pred_len, double* __restrict__ kv_bytes) {
  float p = 0.0f;
  if (tools != 0) {
    const float s = 1.0f / (1.0f + __expf(-(z0 + b_last[0])));
    const int K = tp.n_knots;
    if (!(s > kx[0])) {
      p = ky[0];
    } else if (s >= kx[K - 1]) {
      p = ky[K - 1];
    } else {   // kx[lo] <= s < kx[hi]: the segment through knots lo and lo + 1
      int lo = 0, hi = K - 1;
      while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (kx[mid] <= s) lo = mid;
        else hi = mid;
      }
      p = ky[lo] + (s - kx[lo]) * (ky[hi] - ky[lo]) / (kx[hi] - kx[lo]);
    }
  }
  const float y = zg + b_last[g] + coef[g] * p;
  const float L = fminf(expm1f(fmaxf(y, 0.0f)), tp.max_len);
  if (tp.p_tool) tp.p_tool[row] = p;
  pred_len[row] = L;
  kv_bytes[row] = ((double)prompt + (double)L) * alpha_of(alpha, model, n_models);
}

// Per-role regressors (Sec. III-B): a stage whose role has a regressor of its own is predicted by
// that regressor's network; output 0 regresses log(1 + L), fed the first phase's calibrated tool
// probability p: L = min(expm1(max(z_0 + coef p, 0)), max_len), then Eq. 3. Stages reach the
// kernel bucketed by regressor (every tile belongs to one), in tile-row order, with their stage
// index, prompt length, model id and p carried alongside; padding rows have stage -1.
__device__ __forceinline__ void role_row(float z0, float b0, float coef, float p, float max_len, int32_t stage,
                                         int32_t prompt, int32_t model, const float* __restrict__ alpha,
                                         int32_t n_models, float* __restrict__ pred_len,
                                         double* __restrict__ kv_bytes) {
  const float y = z0 + b0 + coef * p;
  const float L = fminf(expm1f(fmaxf(y, 0.0f)), max_len);
  pred_len[stage] = L;
  kv_bytes[stage] = ((double)prompt + (double)L) * alpha_of(alpha, model, n_models);
}

// Output neuron (within a 32-neuron block) computed by row i of a weight tile. With this order
// the 16 results that lane-half h holds after a 32x32 MFMA (register v -> tile row
// (v/4)*8 + 4h + v%4) are the neurons 16*(v/8) + 8h + v%8: two runs of 8 consecutive
// neurons, which the next layer consumes in natural column order.
__device__ __forceinline__ int tile_row_neuron(int i) {
  const int q = i >> 3;
  return 16 * (q >> 1) + 8 * ((i >> 2) & 1) + 4 * (q & 1) + (i & 3);
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Accumulator of a 32-neuron block initialised with the biases of the neurons lane-half h holds
// (registers 0-7: neurons 8h .. 8h+7, registers 8-15: neurons 16+8h .. 16+8h+7).
__device__ __forceinline__ f32x16 bias_acc(const float* __restrict__ b32, int h) {
  const float4 q0 = *reinterpret_cast<const float4*>(b32 + 8 * h);
  const float4 q1 = *reinterpret_cast<const float4*>(b32 + 8 * h + 4);
  const float4 q2 = *reinterpret_cast<const float4*>(b32 + 16 + 8 * h);
  const float4 q3 = *reinterpret_cast<const float4*>(b32 + 16 + 8 * h + 4);
  return f32x16{q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w,
                q2.x, q2.y, q2.z, q2.w, q3.x, q3.y, q3.z, q3.w};
}

typedef short s16x2 __attribute__((ext_vector_type(2)));

// acc[8*half + j] (biases included), j = 0..7, rounded to bfloat16 (nearest even) and packed as
// the 8 K-slots of a B operand, then rectified on the packed values: a bfloat16 is below zero
// exactly when its bit pattern is a negative int16, so a packed int16 max with 0 is the ReLU
// (rounding to nearest and ReLU commute; -0 becomes +0).
__device__ __forceinline__ bf16x8 relu_bf16(const f32x16& acc, int half) {
  uint32_t w[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const f32x2 f = {acc[8 * half + 2 * p], acc[8 * half + 2 * p + 1]};
    const s16x2 v = __builtin_bit_cast(s16x2, __builtin_convertvector(f, bf16x2));
    w[p] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(v, s16x2{0, 0}));
  }
  return __builtin_bit_cast(bf16x8, make_uint4(w[0], w[1], w[2], w[3]));
}

// Direct global->LDS loads through a raw buffer resource: lane l's 16 (or 4) bytes at byte offset
// voff + soff of the buffer land at LDS byte address lds_base + lds_off + 16 l (or 4 l). Without soff,
// lanes whose voff is at or past the buffer's size read zeros and touch no memory; a load that may pass
// the buffer's end therefore carries its whole offset in voff (dma16_once, dma4: the outcome of a size
// smaller than soff is not defined), and soff is for loads that stay inside the buffer. Issued as inline
// assembly so that the compiler's automatic wait insertion, which would conservatively drain
// every such load before any LDS read, does not see them; the kernel waits for them itself
// (wait_chunk). rsrc, soff and lds_base are wavefront-uniform; lds_off is a compile-time constant.
// An LDS-DMA load reads M0 and needs one wait state after the scalar write of M0 (a hazard the
// compiler resolves only for instructions it generates itself), hence the s_nop.
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) unsigned char lds_uchar;

// Raw (unstrided) buffer resource over `bytes` bytes at `base` (gfx9 descriptor: 48-bit base,
// stride 0, byte-granular range check, 32-bit data format).
__device__ __forceinline__ i32x4 buffer_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int32_t)((a >> 32) & 0xFFFF));
  r[2] = __builtin_amdgcn_readfirstlane((int32_t)bytes);
  r[3] = 0x00020000;
  return r;
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const lds_uchar*)(p);
}
__device__ __forceinline__ void dma16(const i32x4& rsrc, uint32_t voff, uint32_t soff, uint32_t lds_base,
                                      int lds_off) {
  asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, %4 offen lds"
               ::"s"(lds_base), "i"(lds_off), "v"(voff), "s"(rsrc), "s"(soff) : "m0", "scc");
}
// For data read once (features, per-stage inputs), which may pass the buffer's end: no scalar offset,
// and non-temporal (nt), a candidate for early eviction that does not push the weights, which every
// tile re-reads, out of the L2 cache.
__device__ __forceinline__ void dma16_once(const i32x4& rsrc, uint32_t voff, uint32_t lds_base, int lds_off) {
  asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen nt lds"
               ::"s"(lds_base), "i"(lds_off), "v"(voff), "s"(rsrc) : "m0", "scc");
}
__device__ __forceinline__ void dma4(const i32x4& rsrc, uint32_t voff, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen nt lds"
               ::"s"(lds_base), "v"(voff), "s"(rsrc) : "m0");
}

constexpr int kMaxModels = 64;           // per-model KV bytes staged in LDS

}  // namespace maestro
