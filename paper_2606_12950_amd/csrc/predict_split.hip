// The bfloat16 predictor for small batches: a workgroup's four wavefronts split the neurons of a
// layer instead of the rows.
//
// The large-batch kernel gives every wavefront 32 or 64 rows and streams all weights through LDS
// once per 128- or 256-row tile, which the rows of the tile share. A batch of fewer tiles than
// compute units leaves the chip partly idle and still takes a whole tile's time (31 us for the
// 512-wide network, 50 us for the 1024-wide one). Here a tile is one or two groups of 32 rows, so
// that the same batch spreads over 4 times as many compute units. Every wavefront holds the
// layer-1 activations of all rows of the tile (256 accumulation registers) and computes a quarter of
// the 32-neuron blocks, streaming just those blocks' weights through an LDS ring of its own: no
// barrier and no sharing inside a layer. Between layers the wavefronts exchange their activations
// through LDS, half a layer at a time, which leaves the LDS to the rings (28 KB each, 24 KB of loads
// in flight per wavefront).
//
// What bounds a tile: the stream of all weights through one compute unit, 0.85 or 2.6 MB at about 47
// bytes per clock, and about 8 us of features, exchanges and epilogue. Measured: 17.7 us (512-wide) and
// 33 us (1024-wide) for up to one tile per compute unit. The chunk fetched next comes from a table
// in LDS rather than from index arithmetic (which took the 1024-wide tile to 118 us, one wavefront
// per SIMD having nothing to hide it behind), and the loops over blocks stay rolled: unrolled they
// took 100 KB of code and no less time (35 us).
//
// Every sum is taken over the same inputs in the same order as in the large-batch kernel (32x32x16
// MFMAs over 16 consecutive inputs at a time, accumulators started from the biases, output sums
// over ascending blocks), so a stage's prediction has the same bits whichever kernel ran.
#include <type_traits>

#include "feature_load.h"
#include "internal.h"
#include "mlp.h"

namespace maestro {
namespace {

enum SplitMode { kBins = 0, kTwoPhaseHeads = 1, kRoleRegressors = 2 };

struct SplitArgs {
  const uint16_t *x, *w1, *w2, *w3;
  const float *b1, *b2, *b3, *centre;     // centre: bins only
  int64_t n;
  const int32_t *prompt_len, *model_id;   // per stage, or per tile row (role regressors)
  const float* alpha;
  int32_t n_models;
  float* pred_len;
  double* kv_bytes;
  TwoPhaseArgs tp;
  const int32_t *group_tile, *perm, *p_bits;   // role regressors: tile count and first tile of each group
  int32_t n_groups;
  const float* role_coef;
  float role_max_len;
};

constexpr int kD = 256, kB = 64;
constexpr int kSplitThreads = 256;
constexpr int kChunk = 4096;             // 32 weight rows x 64 inputs: four K-steps
constexpr int kSlots = 7;                // chunks of a wavefront's ring
constexpr int kAheadFr = 3;              // fragments read ahead of their MFMA

// Wavefront-level waits (gfx9 s_waitcnt encoding: vmcnt in bits 3:0 and 15:14, lgkmcnt in 11:8).
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
  asm volatile("" ::: "memory");
}
// workgroup barrier after this wavefront's LDS accesses, leaving its loads in flight
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4) | (0 << 8));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int H, int G, int kMode>
__global__ __launch_bounds__(kSplitThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
void mlp3_split_kernel(const SplitArgs a) {
  constexpr int R = 32 * G;              // rows of a tile
  constexpr int KS1 = kD / 16, KS2 = H / 16, KSH = KS2 / 2;
  constexpr int HB = H / 64;             // 32-neuron blocks of half a layer
  constexpr int PW = HB / 4;             // of which each wavefront takes PW: block 4 i + wave
  constexpr int C1 = kD / 64, C2 = H / 64, C3 = KSH / 4;   // chunks of a layer-1 / layer-2 block, of half of W3
  constexpr int kActBytes = G * KSH * 1024;
  // chunks of a wavefront's stream, and the empty ones that its prefetch runs into
  constexpr int kStream = 2 * PW * C1 + 2 * (PW * C2 + C3) + kSlots;
  static_assert(kActBytes >= R * kD * 2, "the features share the exchange buffer");
  constexpr bool kRoles = kMode == kRoleRegressors, kTwo = kMode == kTwoPhaseHeads;

  // features of the tile, then half a layer's activations at a time: fragment (group, K-step) of
  // 64 lanes x 16 bytes, exactly the B operand each lane feeds
  __shared__ __attribute__((aligned(16))) unsigned char s_act[kActBytes];
  __shared__ __attribute__((aligned(16))) unsigned char s_ring[4][kSlots * kChunk];
  __shared__ __attribute__((aligned(16))) float s_b1[H], s_b2[H], s_b3[64], s_c[64], s_alpha[64];
  __shared__ __attribute__((aligned(16))) int32_t s_meta[4][64];
  __shared__ __attribute__((aligned(16))) int32_t s_head[kTwo ? 64 : 1];
  __shared__ __attribute__((aligned(16))) float s_kx[kTwo ? 64 : 1], s_ky[kTwo ? 64 : 1];
  __shared__ uint32_t s_stream[4][kStream];   // what each wavefront fetches, chunk by chunk

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63, h = lane >> 5, r32 = lane & 31;
  const int64_t tile = blockIdx.x;

  // this tile's regressor: the last group whose first tile is not past it
  int grp = 0;
  if constexpr (kRoles) {
    if (tile >= a.group_tile[0]) return;   // whole workgroups: past the last tile
    for (int g = 1; g < a.n_groups; ++g) grp = tile >= a.group_tile[1 + g] ? g : grp;
    grp = __builtin_amdgcn_readfirstlane(grp);
  }
  const i32x4 rs1 = buffer_rsrc(a.w1 + (size_t)grp * (H * kD), H * kD * 2);
  const i32x4 rs2 = buffer_rsrc(a.w2 + (size_t)grp * (H * H), H * H * 2);
  const i32x4 rs3 = buffer_rsrc(a.w3 + (size_t)grp * (kB * H), kB * H * 2);

  // ---- the tile's inputs: direct loads into LDS
  const int64_t row0 = tile * R;
  const uint32_t rows = kRoles ? (uint32_t)R : (uint32_t)(a.n - row0 < R ? a.n - row0 : R);
  {
    // feature load q: rows 2i (lanes 0-31) and 2i + 1, i = wave + 4q (feature_load.h)
    const uint32_t base = lds_addr(s_act) + wave * 1024;
    if constexpr (kRoles) {
      const i32x4 rs = buffer_rsrc(a.x, (uint32_t)(a.n * (kD * 2)));
      int32_t st[R / 8];
#pragma unroll
      for (int q = 0; q < R / 8; ++q) st[q] = a.perm[row0 + 2 * (wave + 4 * q) + h];
#pragma unroll
      for (int q = 0; q < R / 8; ++q) {
        const uint32_t unit = (uint32_t)(((lane & 31) ^ ((2 * (wave + 4 * q) + h) & 15)) << 4);
        dma16_once(rs, st[q] >= 0 ? (uint32_t)st[q] * (uint32_t)(kD * 2) + unit : 0x80000000u, base, q * 4096);
      }
    } else {
      const i32x4 rs = buffer_rsrc(a.x + row0 * kD, rows * kFeatureRow);
#pragma unroll
      for (int q = 0; q < R / 8; ++q) dma16_once(rs, feature_offset_split(q, wave, lane), base, q * 4096);
    }
    const i32x4 rb1 = buffer_rsrc(a.b1 + (size_t)grp * H, H * 4), rb2 = buffer_rsrc(a.b2 + (size_t)grp * H, H * 4);
    for (int i = wave; i < H / 256; i += 4) {
      dma16(rb1, (uint32_t)(lane * 16), (uint32_t)(i * 1024), lds_addr(s_b1) + i * 1024, 0);
      dma16(rb2, (uint32_t)(lane * 16), (uint32_t)(i * 1024), lds_addr(s_b2) + i * 1024, 0);
    }
    const uint32_t v4 = (uint32_t)(lane * 4);
    if (wave == 0) {
      dma4(buffer_rsrc(a.b3 + (size_t)grp * kB, kB * 4), v4, lds_addr(s_b3));
      dma4(buffer_rsrc(a.alpha, (uint32_t)a.n_models * 4), v4, lds_addr(s_alpha));
      if constexpr (kTwo) dma4(buffer_rsrc(a.tp.role_head, (uint32_t)a.tp.n_roles * 4), v4, lds_addr(s_head));
    } else if (wave == 1) {
      if constexpr (!kRoles) dma4(buffer_rsrc(kTwo ? a.tp.tool_coef : a.centre, kB * 4), v4, lds_addr(s_c));
      if constexpr (kTwo) {
        dma4(buffer_rsrc(a.tp.iso_x, (uint32_t)a.tp.n_knots * 4), v4, lds_addr(s_kx));
        dma4(buffer_rsrc(a.tp.iso_y, (uint32_t)a.tp.n_knots * 4), v4, lds_addr(s_ky));
      }
    } else if (wave == 2) {
      dma4(buffer_rsrc(a.prompt_len + row0, rows * 4), v4, lds_addr(s_meta[0]));
      dma4(buffer_rsrc(a.model_id + row0, rows * 4), v4, lds_addr(s_meta[1]));
    } else {
      if constexpr (kMode != kBins) {
        dma4(buffer_rsrc((kRoles ? a.p_bits : a.tp.role_id) + row0, rows * 4), v4, lds_addr(s_meta[2]));
        dma4(buffer_rsrc((kRoles ? a.perm : a.tp.tool_avail) + row0, rows * 4), v4, lds_addr(s_meta[3]));
      }
    }
  }

  // ---- this wavefront's weight stream: W1 blocks of both halves, W2 blocks of the first half, then
  // (wavefronts that sum outputs) the first half of W3's inputs, and the same for the second half.
  // Output wavefronts: group g, outputs 32 bt .. 32 bt + 31 (output 0 alone with role regressors).
  const int og = G == 2 ? wave >> 1 : 0, bt = wave & 1;
  const bool outputs = (G == 2 || wave < 2) && (!kRoles || bt == 0);
  const int n3 = outputs ? C3 : 0;
  const uint32_t ring = lds_addr(s_ring[wave]);
  // piece q of a chunk: rows 8q .. 8q+7 (lane / 8), unit u of row r at u ^ (r/2 % 8)
  const uint32_t lrow = (uint32_t)lane >> 3, unit0 = (uint32_t)(((lane & 7) ^ (lane >> 4)) << 4), unit1 = unit0 ^ 64u;
  // The stream as a table, built by the lanes in parallel: byte offset of a chunk in its matrix, and
  // the matrix in the top bits (0: W1, 1: W2, 2: W3, 3: none -- past the stream's end nothing is read,
  // but the loads still count, so that every wait below is for a fixed number of them).
  for (int e = lane; e < kStream; e += 64) {
    uint32_t v;
    int c = e;
    if (c < 2 * PW * C1) {
      const int blk = c / C1;
      v = (uint32_t)(((blk / PW) * HB + (blk % PW) * 4 + wave) * 32 * kD * 2 + (c % C1) * 128);
    } else {
      c -= 2 * PW * C1;
      const int half = c >= PW * C2 + n3 ? 1 : 0;
      c -= half ? PW * C2 + n3 : 0;
      if (c < PW * C2) v = 1u << 28 | (uint32_t)((half * HB + (c / C2) * 4 + wave) * 32 * H * 2 + (c % C2) * 128);
      else if (c - PW * C2 < n3) v = 2u << 28 | (uint32_t)(32 * bt * H * 2 + half * H + (c - PW * C2) * 128);
      else v = 3u << 28;
    }
    s_stream[wave][e] = v;
  }
  const uint32_t* entry = s_stream[wave];   // of the chunk fetched next
  uint32_t ahead = *entry++;
  struct Load {                            // the chunk whose pieces are going out
    i32x4 rs;
    uint32_t v0, v1, soff, piece;
  };
  auto next_load = [&]() {
    const uint32_t e = __builtin_amdgcn_readfirstlane(ahead);
    ahead = *entry++;
    const uint32_t kind = e >> 28;
    Load l;
#pragma unroll
    for (int i = 0; i < 3; ++i)
      l.rs[i] = __builtin_amdgcn_readfirstlane(kind == 0 ? rs1[i] : kind == 1 ? rs2[i] : i < 2 || kind == 2 ? rs3[i] : 0);
    l.rs[3] = rs1[3];
    l.soff = e & 0x0FFFFFFFu;
    const uint32_t stride = kind == 0 ? kD * 2 : H * 2;
    l.v0 = __umul24(lrow, stride) + unit0;
    l.v1 = __umul24(lrow, stride) + unit1;
    l.piece = 8 * stride;
    return l;
  };
  auto issue = [&](const Load& l, int q, uint32_t dst) { dma16(l.rs, q & 1 ? l.v1 : l.v0, l.soff + q * l.piece, dst, q * 1024); };
#pragma unroll 1
  for (int c = 0; c < kSlots - 1; ++c) {
    const Load l = next_load();
#pragma unroll
    for (int q = 0; q < 4; ++q) issue(l, q, ring + c * kChunk);
  }

  // fragment (K-step kk of a chunk) of this lane: weight rows in the order that leaves a block's
  // results as the next layer's inputs (tile_row_neuron), W3 rows as they are
  const int prow = tile_row_neuron(r32);
  int offw[4], offo[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) {
    offw[kk] = prow * 128 + (((2 * kk + h) ^ ((prow >> 1) & 7)) << 4);
    offo[kk] = r32 * 128 + (((2 * kk + h) ^ ((r32 >> 1) & 7)) << 4);
  }
  // byte offsets in the ring of the chunk being consumed, the next one, and the free slot before it
  const unsigned char* my_ring = s_ring[wave];
  uint32_t slot = 0, slot_next = kChunk, slot_free = (kSlots - 1) * kChunk;
  auto frag = [&](uint32_t s, int off) { return *reinterpret_cast<const bf16x8*>(my_ring + s + off); };
  bf16x8 fr[kAheadFr];
  // the first fragments of a run of blocks (their chunk landed: five later chunks in flight)
  auto prime = [&](const int (&off)[4]) {
    wait_vm<4 * (kSlots - 2)>();
#pragma unroll
    for (int f = 0; f < kAheadFr; ++f) fr[f] = frag(slot, off[f]);
  };
  // KS K-steps of the stream. The slot before the current chunk's is free (its last fragment was
  // consumed), so the chunk six ahead goes there, a piece per step; the next chunk's first fragment
  // is read at step 1 of a chunk, after its loads (17 later ones outstanding: four chunks and one
  // piece).
  auto run = [&](auto ks_tag, const int (&off)[4], auto&& mma) {
    constexpr int KS = decltype(ks_tag)::value;
    static_assert(KS % 4 == 0, "whole chunks");
    Load load;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int pos = ks & 3;
      const bf16x8 f0 = fr[0];
      fr[0] = fr[1];
      fr[1] = fr[2];
      if (pos == 1) wait_vm<4 * (kSlots - 3) + 1>();
      fr[2] = frag(pos == 0 ? slot : slot_next, off[(pos + kAheadFr) & 3]);
      if (pos == 0) load = next_load();
      issue(load, pos, ring + slot_free);
      mma(ks, f0);
      __builtin_amdgcn_sched_barrier(0);
      if (pos == 3) {
        slot_free = slot;
        slot = slot_next;
        slot_next = slot_next == (kSlots - 1) * kChunk ? 0u : slot_next + kChunk;
      }
    }
  };
  auto act = [&](int g, int k) { return reinterpret_cast<bf16x8*>(s_act + ((g * KSH + k) * 64 + lane) * 16); };

  wait_vm<4 * (kSlots - 1)>();             // this wavefront's share of the inputs has landed
  lds_barrier();
  bf16x8 xf[G][KS1];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int ks = 0; ks < KS1; ++ks) {
      const int row = 32 * g + r32;
      xf[g][ks] = *reinterpret_cast<const bf16x8*>(s_act + row * 512 + (((2 * ks + h) ^ (row & 15)) << 4));
    }

  lds_barrier();                           // the exchange buffer is free

  // one 32-neuron block: KS K-steps against the B operands in(g, ks); the results, rectified and
  // rounded, go to the exchange buffer as fragments of block i of the half
  auto block = [&](auto ks_tag, const float* bias, int i, auto&& in) {
    f32x16 acc[G];
#pragma unroll
    for (int g = 0; g < G; ++g) acc[g] = bias_acc(bias, h);
    run(ks_tag, offw, [&](int ks, const bf16x8& f) {
#pragma unroll
      for (int g = 0; g < G; ++g) {
        acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, in(g, ks), acc[g], 0, 0, 0);
        asm volatile("" : "+v"(acc[g]));   // here, among the step's reads and loads
      }
    });
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int half = 0; half < 2; ++half) *act(g, 2 * i + half) = relu_bf16(acc[g], half);
  };
  typedef std::integral_constant<int, KS1> L1;
  typedef std::integral_constant<int, KS2> L2;
  typedef std::integral_constant<int, KSH> L3;

  // ---- layer 1; its activations are held in the accumulation registers
  bf16x8 h1[G][KS2];
  prime(offw);
#pragma unroll
  for (int half = 0; half < 2; ++half) {
#pragma unroll 1
    for (int i = 0; i < PW; ++i)
      block(L1{}, s_b1 + half * (H / 2) + (4 * i + wave) * 32, 4 * i + wave,
            [&](int g, int ks) -> const bf16x8& { return xf[g][ks]; });
    lds_barrier();
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int k = 0; k < KSH; ++k) {
        h1[g][half * KSH + k] = *act(g, k);
        asm volatile("" : "+a"(h1[g][half * KSH + k]));
      }
    lds_barrier();
  }

  // ---- layer 2, and the outputs of each half of it
  f32x16 logit = {};
#pragma unroll 1
  for (int half = 0; half < 2; ++half) {
#pragma unroll 1
    for (int i = 0; i < PW; ++i)
      block(L2{}, s_b2 + half * (H / 2) + (4 * i + wave) * 32, 4 * i + wave,
            [&](int g, int ks) -> const bf16x8& { return h1[g][ks]; });
    lds_barrier();
    if (outputs) {                         // wavefront-uniform
      prime(offo);
      bf16x8 hb[kAheadFr];
#pragma unroll
      for (int f = 0; f < kAheadFr; ++f) hb[f] = *act(og, f);
      run(L3{}, offo, [&](int ks, const bf16x8& f) {
        const bf16x8 b = hb[0];
        hb[0] = hb[1];
        hb[1] = hb[2];
        if (ks + kAheadFr < KSH) hb[2] = *act(og, ks + kAheadFr);
        logit = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, b, logit, 0, 0, 0);
      });
      prime(offw);                         // the second half's first fragments again, in their own order
    }
    lds_barrier();
  }

  // ---- a row's outputs meet in the wavefront of its first 32
  const int local = 32 * og + r32;
  const int64_t row = row0 + local;
  if constexpr (kRoles) {
    if (outputs && h == 0) {
      const int32_t stage = s_meta[3][local];
      if (stage >= 0)
        role_row(logit[0], s_b3[0], a.role_coef[grp], __int_as_float(s_meta[2][local]), a.role_max_len, stage,
                 s_meta[0][local], s_meta[1][local], s_alpha, a.n_models, a.pred_len, a.kv_bytes);
    }
  } else {
    float4* out = reinterpret_cast<float4*>(s_act);
    if (outputs && bt == 1)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        out[(og * 4 + v) * 64 + lane] = make_float4(logit[4 * v], logit[4 * v + 1], logit[4 * v + 2], logit[4 * v + 3]);
    lds_barrier();
    if (outputs && bt == 0) {
      f32x16 z[2];
      z[0] = logit;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float4 f = out[(og * 4 + v) * 64 + lane];
        z[1][4 * v] = f.x;
        z[1][4 * v + 1] = f.y;
        z[1][4 * v + 2] = f.z;
        z[1][4 * v + 3] = f.w;
      }
      if constexpr (kTwo) {
        const int gh = head_of_role(s_meta[2][local], s_head, a.tp.n_roles, kB);
        const float zg = head_output<2>(z, gh, h);
        const float z0 = __shfl(z[0][0], r32);     // output 0: register 0 of lane-half 0
        if (h == 0 && row < a.n)
          two_phase_row(z0, zg, gh, s_b3, s_c, s_kx, s_ky, a.tp, row, s_meta[0][local], s_meta[1][local],
                        s_meta[3][local], s_alpha, a.n_models, a.pred_len, a.kv_bytes);
      } else {
        length_epilogue<2>(z, s_b3, s_c, h, row, a.n, s_meta[0][local], s_meta[1][local], s_alpha, a.n_models,
                           a.pred_len, a.kv_bytes);
      }
    }
  }
  wait_vm<0>();                            // no load into LDS outlives the workgroup
}

template <int kMode>
maestro_status launch_split(const maestro_predictor& p, const SplitArgs& a, int64_t tiles, hipStream_t stream) {
  const dim3 grid((unsigned)tiles), block(kSplitThreads);
  if (p.dims[1] == 512) mlp3_split_kernel<512, 2, kMode><<<grid, block, 0, stream>>>(a);
  else mlp3_split_kernel<1024, 1, kMode><<<grid, block, 0, stream>>>(a);
  return launch_status();
}

SplitArgs split_args(const maestro_predictor& p, int64_t n, const void* x, const int32_t* prompt_len,
                     const int32_t* model_id, const float* alpha, int32_t n_models, float* pred_len,
                     double* kv_bytes) {
  SplitArgs a{};
  a.x = static_cast<const uint16_t*>(x);
  a.w1 = static_cast<const uint16_t*>(p.weight[0]);
  a.w2 = static_cast<const uint16_t*>(p.weight[1]);
  a.w3 = static_cast<const uint16_t*>(p.weight[2]);
  a.b1 = p.bias[0];
  a.b2 = p.bias[1];
  a.b3 = p.bias[2];
  a.n = n;
  a.prompt_len = prompt_len;
  a.model_id = model_id;
  a.alpha = alpha;
  a.n_models = n_models;
  a.pred_len = pred_len;
  a.kv_bytes = kv_bytes;
  return a;
}

}  // namespace

int32_t split_tile_rows(const maestro_predictor& p) { return p.dims[1] == 512 ? 64 : 32; }

maestro_status launch_predict_split(const maestro_predictor& p, const TwoPhaseArgs* tp, int64_t n, const void* x,
                                    const int32_t* prompt_len, const int32_t* model_id,
                                    const float* kv_bytes_per_token, int32_t n_models, float* pred_len,
                                    double* kv_bytes, hipStream_t stream) {
  SplitArgs a = split_args(p, n, x, prompt_len, model_id, kv_bytes_per_token, n_models, pred_len, kv_bytes);
  const int64_t tiles = (n + split_tile_rows(p) - 1) / split_tile_rows(p);
  if (tp) {
    a.tp = *tp;
    return launch_split<kTwoPhaseHeads>(p, a, tiles, stream);
  }
  a.centre = p.bin_centre;
  return launch_split<kBins>(p, a, tiles, stream);
}

maestro_status launch_roles_split(const maestro_predictor& p, int64_t n, const void* x, const float* coef,
                                  float max_len, const int32_t* group_tile, int32_t n_groups, const int32_t* perm,
                                  const int32_t* prompt_p, const int32_t* model_p, const int32_t* p_bits,
                                  int64_t max_tiles, const float* kv_bytes_per_token, int32_t n_models,
                                  float* pred_len, double* kv_bytes, hipStream_t stream) {
  SplitArgs a = split_args(p, n, x, prompt_p, model_p, kv_bytes_per_token, n_models, pred_len, kv_bytes);
  a.group_tile = group_tile;
  a.n_groups = n_groups;
  a.perm = perm;
  a.p_bits = p_bits;
  a.role_coef = coef;
  a.role_max_len = max_len;
  return launch_split<kRoleRegressors>(p, a, max_tiles, stream);
}

}  // namespace maestro
