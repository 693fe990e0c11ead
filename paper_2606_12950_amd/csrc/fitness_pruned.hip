// Routing by fitness (Eq. 5, Alg. 3) without scoring every pair.
//
// A pair's fitness is S = A - pen with A = gamma prox + (1 - gamma) fit, fit = R_need / headroom.
// Everything but the fit depends on the node and on the stage's (class, source, model) alone, and
// the fit falls with the headroom. So the nodes are put in ascending headroom, and for every
// (class, source, model) the largest gamma prox - pen of each block of 8 and of 64 consecutive
// nodes is tabulated: block maximum + (1 - gamma) min(1, R_need / smallest headroom) bounds the
// fitness of every node of the block. A stage scores the sub-blocks of the best bounds first and
// then only the blocks whose bound reaches its k-th best score so far. The scores are the same
// float32 expressions in the same order as in fitness_kernel, the lists are ordered by (score,
// node index), and a block is skipped only when its bound, widened by more than every rounding
// error in it, is below the k-th best, so the outputs are those of scoring every pair.
//
// With degradation plans (Alg. 2, Eq. 4) the nodes that fall short of the demand are the first
// ones in headroom order. Their fit exceeds 1, so they come first: a wavefront goes through
// them together (node data and plan records are then wavefront-uniform), block by block under
// the same bounds, the C_deg term bounded by its smallest value. Where those bounds do not help (all
// nodes short of room, one headroom, plans that fail) every short pair would be looked at, so after a few
// sub-blocks short_pass goes on, with a bound for each node (the cheapest step of its plan, what all its
// steps free) and, in small batches, up to eight wavefronts for the same stages: 8,192 stages on 4,096
// nodes without headroom take 165 us, 796 without short_pass, 168 scoring every pair; 500,000 stages
// 1,650, 2,010 and 1,620; with plans that free little 680, 1,940 and 3,090. (short_pass for all short pairs:
// 47 against 42 us on 512 nodes whose bounds prune well.)
//
// Three launches: ranks of the headrooms and the sorted node records; the penalty, proximity and
// bound tables and the sorted plans; the stages.
// What bounds it: scoring every pair costs 14 vector instructions a pair; here a lane reads up to
// M / 256 float4 of bounds, visits one to five sub-blocks of 8 nodes, and a wavefront waits for
// the lane that visits most, each visit two dependent rounds of divergent 16-byte reads. On 512
// nodes a wavefront takes 1,400 vector instructions (26 us of the kernel's 43 for 719,712 stages,
// 38 of 64 lanes active); on 4,096 nodes 3,900 for its two rounds with plans, and the slowest
// wavefront twice the average one's time.
// Measured (one MI355X, whole call, against scoring every pair): 719,712 stages on 512 nodes, one
// result, 44 .. 49 against 139 us; 500,009 stages on 4,096 nodes with plans, four results, 69
// against 1,150 us. The pass over the 64-node bounds of 4,096 nodes took half of all vector
// instructions (7,200 a wavefront, 88 us) before it ended early. Slower or no faster: plan records
// read eight at a time by the lanes and broadcast (no change), 80 registers for a sixth wavefront
// per SIMD (51 against 43 us on 512 nodes), all tables in LDS with 1,024 lanes a CU (61 against 50
// us a call), sub-block bounds as packed integer keys (no change).
#include "fitness.h"
#include "fitness_grid.h"
#include "internal.h"
#include "select.h"

namespace maestro {
namespace {

constexpr int kThreads = 512;            // of the stage kernel, at most (fitness_grid.h)
constexpr int kMaxNodes = 4096;          // one 64-bit mask of 64-node blocks; node records in LDS
constexpr int kRecSteps = MAESTRO_PLAN_RECORD_STEPS;
// Tied sub-blocks that a stage visits before it leaves the rest to tie_pass: one or two are common among
// 512 nodes without any equal scores (leaving at the first: 58 against 48 us on 719,712 stages).
constexpr int kTies = 2;
// Sub-blocks of nodes that fall short that 64 stages visit before they leave the rest to short_pass, alone
// and where other wavefronts share it. Stages whose bounds prune well visit fewer; nodes without headroom, plans
// that free little (500,000 stages on 512 nodes: 100, 120, 160, 210 us at 8, 16, 32, never) visit up to all.
constexpr int kShortAlone = 16, kShortShared = 4;
constexpr int kMaxGroups = kThreads / 128;   // groups of 64 stages of a workgroup whose wavefronts share
constexpr int kSlots = 2;                // of them, those whose lists meet at a time: little LDS beside the nodes

struct __align__(16) SortedNode {
  double free, recip;                    // headroom and 1 / fl32(headroom) (0 without headroom)
};
struct __align__(16) SortedPlan {        // of a node that falls short
  double reach;                          // a larger demand is past its headroom and all that its plan frees
  float cost;                            // normalised cost of the plan's cheapest step
  float recip;                           // SortedNode::recip, rounded up
};

// All sizes derive from the node count padded to whole 64-node blocks.
struct Tables {
  // nodes, and floats of a bound row: blocks of 64 (padded to four), of 8, then the largest of the 64s from each on
  // ends: the same of the tables of block extremes, blocks of 64 (padded to four), then of 8
  int32_t padded, row, ends;
  size_t nodes, plans, order, tr, prox, nd, gp, pen, bound, gp_top, pen_low, lowest, total;   // byte offsets
};

Tables tables_of(int32_t n_models, int32_t n_nodes, int32_t n_src, int32_t n_classes) {
  Tables t{};
  t.padded = (n_nodes + 63) & ~63;
  t.row = 2 * (((t.padded >> 6) + 3) & ~3) + (t.padded >> 3);
  t.nodes = 0;
  t.plans = t.nodes + (size_t)t.padded * sizeof(SortedNode);
  t.order = t.plans + (size_t)t.padded * sizeof(SortedPlan);
  t.tr = t.order + (size_t)t.padded * sizeof(uint16_t);
  t.prox = t.tr + (size_t)n_models * t.padded * sizeof(float);
  t.nd = t.prox + (size_t)n_src * t.padded * sizeof(float);
  t.gp = t.nd + (size_t)t.padded * sizeof(float);
  t.pen = t.gp + (size_t)n_classes * n_src * t.padded * sizeof(float);
  t.bound = t.pen + (size_t)n_classes * n_models * t.padded * sizeof(float);
  t.ends = (((t.padded >> 6) + 3) & ~3) + (t.padded >> 3);
  t.gp_top = t.bound + (size_t)n_classes * n_src * n_models * t.row * sizeof(float);
  t.pen_low = t.gp_top + (size_t)n_classes * n_src * t.ends * sizeof(float);
  t.lowest = t.pen_low + (size_t)n_classes * n_models * t.ends * sizeof(float);
  t.total = t.lowest + (size_t)t.ends * sizeof(uint16_t);
  return t;
}

// order-preserving map of float64 bits to unsigned; a headroom that is not a number admits no stage and
// comes first, among the nodes that fall short
__device__ __forceinline__ uint64_t double_key(double d) {
  const uint64_t u = __builtin_bit_cast(uint64_t, d);
  return d != d ? 0ull : (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Position of every node in ascending (headroom, index) order by counting: wavefront w of a
// workgroup takes one node, its lanes compare 64 others at a time (LDS), and the ballots add up
// on the scalar unit. 16 nodes per workgroup, so 4,096 nodes spread over 256 workgroups; the M^2
// compares take 8 us there, a third of what a radix sort in one workgroup does. The wavefront then
// writes the node's terms at its position: lane m norm(T_ready) of model m, lane s 1 - norm(RTT)
// from source s, and norm(C_deg).
constexpr int kRankThreads = 1024;
__global__ __launch_bounds__(kRankThreads) void fitness_rank_kernel(int32_t n_nodes, int32_t padded,
                                                                    int32_t n_models, int32_t n_src,
                                                                    const double* __restrict__ free_bytes,
                                                                    const float* __restrict__ queue_ms,
                                                                    const float* __restrict__ act_ms,
                                                                    const uint64_t* __restrict__ resident_mask,
                                                                    const float* __restrict__ act_matrix,
                                                                    const float* __restrict__ deg_ms,
                                                                    const float* __restrict__ rtt_ms,
                                                                    const float* __restrict__ bounds,
                                                                    SortedNode* __restrict__ nodes,
                                                                    uint16_t* __restrict__ order,
                                                                    float* __restrict__ tr, float* __restrict__ prox,
                                                                    float* __restrict__ nd) {
  __shared__ uint64_t s_key[kMaxNodes];
  const int tid = threadIdx.x, lane = tid & 63;
  for (int j = tid; j < padded; j += kRankThreads) s_key[j] = j < n_nodes ? double_key(free_bytes[j]) : ~0ull;
  __syncthreads();
  const int i = blockIdx.x * (kRankThreads / 64) + (tid >> 6);
  if (i >= padded) return;
  if (i >= n_nodes) {                    // padding: admits nothing
    if (lane == 0) {
      nodes[i] = SortedNode{-INFINITY, 0.0};
      order[i] = 0xFFFFu;                // above every node: no tie is decided by it
      nd[i] = 0.0f;
    }
    if (lane < n_models) tr[(size_t)lane * padded + i] = 0.0f;
    if (lane < n_src) prox[(size_t)lane * padded + i] = 0.0f;
    return;
  }
  const uint64_t key = s_key[i];
  // 64-node groups before the node's own count equal keys too, those after it do not (padding
  // holds the largest key and is never below another)
  int rank = 0;
  const int own = i & ~63;
#pragma unroll 4
  for (int j0 = 0; j0 < own; j0 += 64) rank += __popcll(__ballot(s_key[j0 + lane] <= key));
  {
    const uint64_t o = s_key[own + lane];
    rank += __popcll(__ballot(o < key || (o == key && own + lane < i)));
  }
#pragma unroll 4
  for (int j0 = own + 64; j0 < padded; j0 += 64) rank += __popcll(__ballot(s_key[j0 + lane] < key));
  if (lane == 0) {
    const double fr = free_bytes[i];
    const float frf = __double2float_rn(fr);
    nodes[rank] = SortedNode{fr, frf > 0.0f ? __ddiv_rn(1.0, (double)frf) : 0.0};
    order[rank] = (uint16_t)i;
    nd[rank] = deg_ms ? norm01(deg_ms[i], bounds[4], bounds[5]) : 0.0f;
  }
  if (lane < n_models) {
    const float q = queue_ms[i];
    float ready;
    if (act_matrix) ready = __fadd_rn(q, act_matrix[(size_t)i * n_models + lane]);
    else ready = (resident_mask[i] >> lane) & 1u ? __fadd_rn(q, 0.0f) : __fadd_rn(q, act_ms[i]);
    tr[(size_t)lane * padded + rank] = norm01(ready, bounds[2], bounds[3]);
  }
  if (lane < n_src)
    prox[(size_t)lane * padded + rank] = __fsub_rn(1.0f, norm01(rtt_ms[(size_t)lane * n_nodes + i], bounds[0], bounds[1]));
}

// One workgroup per (class, model), and from 513 nodes on per source, eight consecutive sorted nodes
// per thread: their penalties (with plans lambda norm(T_ready) alone, the C_deg term being the
// pair's), the proximity terms gamma (1 - norm(RTT)) (written by model 0's workgroups), and the
// bound rows of the class's (source, model) pairs. With plans the C_deg term is at least
// min(0, mu), since norm() lies in [0, 1].
__device__ __forceinline__ void load8(const float* __restrict__ p, float (&v)[8]) {
  *reinterpret_cast<float4*>(v) = *reinterpret_cast<const float4*>(p);
  *reinterpret_cast<float4*>(v + 4) = *reinterpret_cast<const float4*>(p + 4);
}
__device__ __forceinline__ void store8(float* __restrict__ p, const float (&v)[8]) {
  *reinterpret_cast<float4*>(p) = *reinterpret_cast<const float4*>(v);
  *reinterpret_cast<float4*>(p + 4) = *reinterpret_cast<const float4*>(v + 4);
}

// Whether a stage's pass over the 64-node bounds ends early: it costs a visit of the stage's first
// sub-blocks ahead of the pass, more than the pass itself over up to 16 blocks when one node is wanted.
__host__ __device__ constexpr bool early_end(int32_t padded) { return padded > 1024; }

// What the plans of nodes in sorted order free and cost at best, eight lanes a node: lane e takes step e of the
// record and every eighth step past it. Workgroup w of n_w.
__device__ __forceinline__ void sort_plans(int w, int n_w, int32_t n_nodes, const SortedNode* __restrict__ nodes,
                                           const uint16_t* __restrict__ order,
                                           const maestro_deg_plan* __restrict__ plans,
                                           const maestro_plan_step* __restrict__ plan_steps, float lo_d, float hi_d,
                                           SortedPlan* __restrict__ sorted_plans) {
  static_assert(kRecSteps == 8, "a step a lane");
  const int per_w = blockDim.x >> 3, e = threadIdx.x & 7;
  for (int p = w * per_w + (int)(threadIdx.x >> 3); p < n_nodes; p += n_w * per_w) {   // the same for the eight lanes
    const maestro_deg_plan& pl = plans[order[p]];
    const SortedNode nd = nodes[p];
    const int ne = pl.n_engines;
    double freed = __shfl(pl.freed[e], min(max(ne, 1), kRecSteps) - 1, 8);
    float cost = pl.cost[e];
    if (e >= ne) cost = INFINITY;
    if (ne > kRecSteps) {
      const maestro_plan_step* st = plan_steps + pl.first_step;
      freed = st[ne - 1].freed;
#pragma unroll 4
      for (int q = kRecSteps + e; q < ne; q += 8) cost = fminf(cost, st[q].cost);
    }
#pragma unroll
    for (int off = 1; off < 8; off <<= 1) cost = fminf(cost, __shfl_xor(cost, off));
    // past every rounding of R_need - headroom, which a stage compares with the freed bytes
    const double slack = (fabs(nd.free) + fabs(freed)) * 0x1p-50;
    if (e == 0)
      sorted_plans[p] = SortedPlan{ne > 0 ? nd.free + freed + slack : -INFINITY, norm01(cost, lo_d, hi_d),
                                   __double2float_ru(nd.recip)};
  }
}

// Rows of workgroups beside those of the classes that take the plans: the reads of a plan, one after another,
// take as long as a table's. (By the rank kernel, which leaves nothing idle: 0.3 us more on 512 nodes, 1.0 on 4,096.)
constexpr int kPlanRows = 8;
template <bool kPlans>
__global__ __launch_bounds__(kMaxNodes / 8) void fitness_tables_kernel(
    int32_t n_models, int32_t n_nodes, int32_t n_src, int32_t padded, int32_t row, const float* __restrict__ tr,
    const float* __restrict__ prox, const float* __restrict__ nd, const float* __restrict__ class_weights,
    const uint16_t* __restrict__ order, float* __restrict__ gp, float* __restrict__ pen, float* __restrict__ bound,
    int32_t ends, float* __restrict__ gp_top, float* __restrict__ pen_low, uint16_t* __restrict__ lowest,
    const SortedNode* __restrict__ nodes, const maestro_deg_plan* __restrict__ plans,
    const maestro_plan_step* __restrict__ plan_steps, const float* __restrict__ bounds,
    SortedPlan* __restrict__ sorted_plans) {
  if constexpr (kPlans) {                // whole workgroups
    const int r = (int)blockIdx.y - ((int)gridDim.y - kPlanRows);
    if (r >= 0) {
      sort_plans((r * gridDim.z + blockIdx.z) * gridDim.x + blockIdx.x, kPlanRows * gridDim.z * gridDim.x, n_nodes, nodes,
                 order, plans, plan_steps, bounds[4], bounds[5], sorted_plans);
      return;
    }
  }
  __shared__ float s_top[64];
  const int m = blockIdx.x, c = blockIdx.y;
  const int p0 = threadIdx.x * 8;        // blockDim.x is padded / 8
  const float gamma = class_weights[3 * c], lambda = class_weights[3 * c + 1], mu = class_weights[3 * c + 2];
  const float deg_floor = fminf(mu, 0.0f);
  float pn[8], low[8], t[8], d[8];
  load8(tr + (size_t)m * padded + p0, t);
  load8(nd + p0, d);
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const float lt = __fmul_rn(lambda, t[u]);
    pn[u] = kPlans ? lt : __fadd_rn(lt, __fmul_rn(mu, d[u]));
    low[u] = p0 + u >= n_nodes ? INFINITY : kPlans ? lt + deg_floor : pn[u];   // padding: bound -inf
  }
  const int blocks4 = ((padded >> 6) + 3) & ~3;
  // the extreme `v` of these eight nodes and, over eight threads, of their block of 64
  auto store_ends = [&](auto* __restrict__ to, auto v, auto&& of) {
    to[blocks4 + (p0 >> 3)] = v;
    v = of(v, __shfl_xor(v, 1));
    v = of(v, __shfl_xor(v, 2));
    v = of(v, __shfl_xor(v, 4));
    if ((threadIdx.x & 7) == 0) to[p0 >> 6] = v;
  };
  if (blockIdx.z == 0) {
    float least = INFINITY;
#pragma unroll
    for (int u = 0; u < 8; ++u) least = p0 + u < n_nodes ? fminf(least, pn[u]) : least;
    store8(pen + (size_t)(c * n_models + m) * padded + p0, pn);
    store_ends(pen_low + (size_t)(c * n_models + m) * ends, least, [](float a, float b) { return fminf(a, b); });
    if (m == 0 && c == 0) {
      const uint4 o = *reinterpret_cast<const uint4*>(order + p0);
      const uint32_t ow[4] = {o.x, o.y, o.z, o.w};
      int least_node = 0xFFFF;
#pragma unroll
      for (int u = 0; u < 8; ++u) least_node = min(least_node, (int)((ow[u >> 1] >> (16 * (u & 1))) & 0xFFFFu));
      store_ends(lowest, least_node, [](int a, int b) { return min(a, b); });
    }
  }
  for (int s = blockIdx.z; s < n_src; s += gridDim.z) {    // workgroup-uniform
    float g[8], top = -INFINITY;
    load8(prox + (size_t)s * padded + p0, g);
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      g[u] = __fmul_rn(gamma, g[u]);
      top = fmaxf(top, g[u] - low[u]);
    }
    if (m == 0) {
      float most = -INFINITY;
#pragma unroll
      for (int u = 0; u < 8; ++u) most = p0 + u < n_nodes ? fmaxf(most, g[u]) : most;
      store8(gp + (size_t)(c * n_src + s) * padded + p0, g);
      store_ends(gp_top + (size_t)(c * n_src + s) * ends, most, [](float a, float b) { return fmaxf(a, b); });
    }
    float* r = bound + (size_t)((c * n_src + s) * n_models + m) * row;
    r[blocks4 + (p0 >> 3)] = top;
    top = fmaxf(top, __shfl_xor(top, 1));
    top = fmaxf(top, __shfl_xor(top, 2));
    top = fmaxf(top, __shfl_xor(top, 4));
    if ((threadIdx.x & 7) == 0) r[p0 >> 6] = top;
    if (early_end(padded)) {               // the largest entry of each block of 64 and those after it
      if ((threadIdx.x & 7) == 0) s_top[p0 >> 6] = top;
      __syncthreads();
      if (threadIdx.x < 64) {              // a whole wavefront: padded exceeds 1,024
        const int lane = threadIdx.x;
        float v = lane < (padded >> 6) ? s_top[lane] : -INFINITY;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const float w = __shfl_down(v, off);
          if (lane + off < 64) v = fmaxf(v, w);
        }
        if (lane < blocks4) r[blocks4 + (padded >> 3) + lane] = v;
      }
      __syncthreads();
    }
  }
}

// Relative widening of the bounds: a score takes four rounded float32 operations on terms no
// larger than |gamma|, (1 - gamma) fit, |lambda| and |mu|, and a bound (from above or below) four,
// so 2^-19 of the sum of those terms is more than all of their rounding errors together (each less
// than 2^-21 of it).
constexpr float kSlack = 1.9073486328125e-06f;

// Plans of a wavefront-uniform node, read by scalar loads. By vector loads, which the compiler takes where it
// does not see that nothing writes there: 46.2 against 44.8 us on 582 nodes, 8,192 stages that are short of room on
// all of 4,096 nodes 340 against 257.
typedef const __attribute__((address_space(4))) maestro_deg_plan* ScalarPlans;
typedef const __attribute__((address_space(4))) SortedPlan* ScalarSortedPlans;

struct WalkArgs {
  int64_t n;
  const int32_t *model_id, *src_id, *class_id;
  const double* kv_bytes;
  int32_t n_models, n_nodes, n_src, n_classes, padded, row;
  const SortedNode* nodes;
  const uint16_t* order;
  const float *gp, *pen, *bound;
  int32_t ends;
  const float *gp_top, *pen_low;
  const uint16_t* lowest;
  const SortedPlan* sorted_plans;
  const maestro_deg_plan* plans;
  const maestro_plan_step* plan_steps;
  const float *class_weights, *bounds;
  double rho;
  int32_t k, parts, merge_at;
  int32_t* node_idx;
  float* fitness;
};

// The kernel's argument, read again where it is used: held from the kernel's start, the pointers of the passes
// that few stages take (and with plans those of a round) fill the scalar registers, and the loops that every stage
// takes spill to vector lanes. On 512 nodes 7% more vector instructions: 56.3 against 54.3 us with plans, 50.3
// against 49.4 without.
typedef const __attribute__((address_space(4))) WalkArgs* ColdArgs;
__device__ __forceinline__ ColdArgs cold_args() {
  ColdArgs p = (ColdArgs)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// What a round of stages reads. With plans it is read again for each round and for the round's end; without
// them it fits the scalar registers (49.1 against 49.9 us on 512 nodes).
struct RoundArgs {
  int64_t n;
  const int32_t *model_id, *src_id, *class_id;
  const double* kv_bytes;
  const float *class_weights, *gp, *pen, *bound;
  int32_t n_models, n_src, n_classes, k;
  double rho;
  int32_t* node_idx;
  float* fitness;
};
template <class Args>
__device__ __forceinline__ RoundArgs round_args(Args a) {
  return RoundArgs{a->n, a->model_id, a->src_id, a->class_id, a->kv_bytes, a->class_weights, a->gp, a->pen, a->bound,
                   a->n_models, a->n_src, a->n_classes, a->k, a->rho, a->node_idx, a->fitness};
}

// Node records of a workgroup in LDS.
struct WalkLds {
  double *free, *recip;                  // [padded]
  float *r8, *r64;                       // [padded / 8], [padded / 64, to a multiple of four]
  uint16_t* order;                       // [padded]
};
__device__ __forceinline__ WalkLds walk_lds(unsigned char* raw, int32_t padded) {
  WalkLds l;
  l.free = reinterpret_cast<double*>(raw);
  l.recip = l.free + padded;
  l.r8 = reinterpret_cast<float*>(l.recip + padded);
  l.r64 = l.r8 + (padded >> 3);
  l.order = reinterpret_cast<uint16_t*>(l.r64 + (((padded >> 6) + 3) & ~3));
  return l;
}

// The rest of a stage whose k-th best score so far ties with the bounds of blocks it has not visited:
// all its blocks again, in sorted order. A block is left out when its bound is below that score, or when
// no node of it can enter the list: its scores are at most the one of the block's largest proximity
// term, its least penalty and the fit on its first admitting node, evaluated as scores are (every
// rounded operation is monotone, so no widening), and on that score only a lower node index enters. Where
// one score fills the list, all blocks but those of lower indices go that way: 719,712 stages on 512
// idle nodes of one kind (one result) take 78 us a call, 131,072 on 4,096 take 68, against 466 and 692
// with every tie visited, and 150 and 400 scoring every pair. Apart from the loops that every stage
// takes, whose registers decide how many wavefronts run (tests inside those loops: 51 against 48 us on
// 719,712 stages without ties), so the stage's inputs are read again.
template <int KT, bool kPlans>
__device__ __forceinline__ void tie_pass(TopK<KT>& best, int64_t stage, int start, unsigned char* raw) {
  const ColdArgs args = cold_args();
  const int32_t n_models = args->n_models, n_nodes = args->n_nodes, n_src = args->n_src, padded = args->padded,
                row = args->row, ends = args->ends;
  const int32_t *model_id = args->model_id, *src_id = args->src_id, *class_id = args->class_id;
  const double *kv_bytes = args->kv_bytes, rho = args->rho;
  const float *gp = args->gp, *pen = args->pen, *bound = args->bound, *gp_top = args->gp_top,
              *pen_low = args->pen_low, *class_weights = args->class_weights, *bounds = args->bounds;
  const uint16_t* lowest = args->lowest;
  const float nd_fits = norm01(0.0f, bounds[4], bounds[5]);
  const WalkLds lds = walk_lds(raw, padded);
  const double* s_recip = lds.recip;
  const float *s_r8 = lds.r8, *s_r64 = lds.r64;
  const uint16_t* s_order = lds.order;
  asm volatile("" : "+v"(stage));          // not the values held since the stage's start
  const int32_t m = model_id[stage], si = src_id[stage], ci = class_id[stage];
  const double need = (rho == 0.0) ? kv_bytes[stage] : __dmul_rn(kv_bytes[stage], 1.0 + rho);
  const double needd = (double)__double2float_rn(need);
  const float gamma = class_weights[3 * ci], lambda = class_weights[3 * ci + 1], mu = class_weights[3 * ci + 2];
  const float omg = __fsub_rn(1.0f, gamma), md = __fmul_rn(mu, nd_fits);
  const float needf = fmaxf((float)needd, 0.0f), fit_w = fmaxf(omg, 0.0f) * (1.0f + kSlack);
  const float widen = (needd < 0.0 && omg < 0.0f)
                          ? INFINITY
                          : kSlack * (fabsf(gamma) + fabsf(lambda) + fabsf(mu) + fabsf(omg));
  const bool monotone = needd >= 0.0 && omg >= 0.0f;   // of the fit; otherwise no block is shut
  const int cs = ci * n_src + si, cm = ci * n_models + m;
  const int blocks = padded >> 6, blocks4 = (blocks + 3) & ~3;
  const float* t64 = bound + ((size_t)cs * n_models + m) * row;
  const float *g64 = gp_top + (size_t)cs * ends, *p64 = pen_low + (size_t)cm * ends;
  auto shut = [&](float ub, float g, float p, int first, int low) {
    const float fit = __double2float_rn(__dmul_rn(needd, s_recip[max(first, start)]));
    const float key = -__fsub_rn(__fadd_rn(g, __fmul_rn(omg, fit)), kPlans ? __fadd_rn(p, md) : p);
    const float kth = best.s[KT - 1];
    return ub < -kth - widen || (monotone && (key > kth || (key == kth && low > best.n[KT - 1])));
  };
  // those of entries q .. q + 3 of a row (blocks of 64, or at + q sub-blocks) that are not shut
  auto open4 = [&](int at, int q, int width, const float* s_r) {
    const float4 t = *reinterpret_cast<const float4*>(t64 + at + q), r = *reinterpret_cast<const float4*>(s_r + q);
    const float4 g = *reinterpret_cast<const float4*>(g64 + at + q), p = *reinterpret_cast<const float4*>(p64 + at + q);
    const uint2 o = *reinterpret_cast<const uint2*>(lowest + at + q);
    const float tv[4] = {t.x, t.y, t.z, t.w}, rv[4] = {r.x, r.y, r.z, r.w}, gv[4] = {g.x, g.y, g.z, g.w},
                pv[4] = {p.x, p.y, p.z, p.w};
    uint32_t mask = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t low = ((u < 2 ? o.x : o.y) >> (16 * (u & 1))) & 0xFFFFu;
      const bool in = (q + u + 1) * width > start && (q + u) * width < n_nodes;
      if (in && !shut(fmaf(fit_w, fminf(needf * rv[u], 1.0f), tv[u]), gv[u], pv[u], (q + u) * width, low)) mask |= 1u << u;
    }
    return mask;
  };
#pragma unroll 1
  for (int q = (start >> 6) & ~3; q < blocks; q += 4) {
#pragma unroll 1
    for (uint32_t m64 = open4(0, q, 64, s_r64); m64; m64 &= m64 - 1) {
      const int blk = q + __ffs(m64) - 1;
#pragma unroll 1
      for (int h = 8 * blk; h < 8 * blk + 8; h += 4) {
#pragma unroll 1
        for (uint32_t m8 = open4(blocks4, h, 8, s_r8); m8; m8 &= m8 - 1) {
          const int i0 = 8 * (h + __ffs(m8) - 1);
          float g[8], l[8];
          load8(gp + (size_t)cs * padded + i0, g);
          load8(pen + (size_t)cm * padded + i0, l);
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            const int i = i0 + u;
            const float fit = __double2float_rn(__dmul_rn(needd, s_recip[i]));
            const float a = __fadd_rn(g[u], __fmul_rn(omg, fit));
            const int32_t node = s_order[i];
            bool take = i >= start && i < n_nodes;
#pragma unroll
            for (int t = 0; t < KT; ++t) take = take && best.n[t] != node;   // scored before
            if (take) best.push_lex(-__fsub_rn(a, kPlans ? __fadd_rn(l[u], md) : l[u]), node);
          }
        }
      }
    }
  }
}

// C_deg of the shortfall R by one node's plan (wavefront-uniform): the cost of the first step that has
// freed R; false where none has. go: the lanes that need it.
__device__ __forceinline__ bool plan_cost(ScalarPlans pl, const maestro_plan_step* __restrict__ plan_steps, double R,
                                          bool go, float& cost) {
  const int ne = pl->n_engines;
  int jp = 0;
#pragma unroll
  for (int e = 0; e < kRecSteps; ++e) jp += pl->freed[e] < R ? 1 : 0;
  cost = pl->cost[0];
#pragma unroll
  for (int e = 1; e < kRecSteps; ++e) cost = jp == e ? pl->cost[e] : cost;
  bool found = jp < ne && jp < kRecSteps;
  if (go && !found && ne > kRecSteps) {    // the steps past the record
    const maestro_plan_step* st = plan_steps + pl->first_step;
    int lo = kRecSteps, hi = ne;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (st[mid].freed < R) lo = mid + 1;
      else hi = mid;
    }
    found = lo < ne;
    if (found) cost = st[lo].cost;
  }
  return found;
}

// The short pairs of 64 stages from sub-block `rest` on, for stages whose bounds prune little: part
// `part` of `parts` wavefronts, which tell each other their k-th best scores (that of the stage is not below
// any of them). A node is looked up only if the cheapest step of its plan can enter the list and all its
// steps free enough. `mine`: the stage's short nodes, 0 without a stage. Reads the stage again, as tie_pass.
template <int KT>
__device__ __forceinline__ void short_pass(TopK<KT>& best, int64_t stage, int mine, int rest, int part, int parts,
                                           uint32_t* floors, unsigned char* raw) {
  const ColdArgs args = cold_args();
  const int32_t n_models = args->n_models, n_src = args->n_src, padded = args->padded, row = args->row;
  const int32_t *model_id = args->model_id, *src_id = args->src_id, *class_id = args->class_id;
  const double *kv_bytes = args->kv_bytes, rho = args->rho;
  const float *gp = args->gp, *pen = args->pen, *bound = args->bound, *class_weights = args->class_weights;
  const ScalarPlans plans = (ScalarPlans)args->plans;
  const ScalarSortedPlans sorted_plans = (ScalarSortedPlans)args->sorted_plans;
  const maestro_plan_step* plan_steps = args->plan_steps;
  const float lo_d = args->bounds[4], hi_d = args->bounds[5];
  const WalkLds lds = walk_lds(raw, padded);
  const double *s_free = lds.free, *s_recip = lds.recip;
  const float *s_r8 = lds.r8, *s_r64 = lds.r64;
  const uint16_t* s_order = lds.order;
  asm volatile("" : "+v"(stage));
  int32_t m = 0, si = 0, ci = 0;
  double need = 0.0;
  if (mine > 0) {
    m = model_id[stage], si = src_id[stage], ci = class_id[stage];
    need = (rho == 0.0) ? kv_bytes[stage] : __dmul_rn(kv_bytes[stage], 1.0 + rho);
  }
  const double needd = (double)__double2float_rn(need);
  const float gamma = class_weights[3 * ci], lambda = class_weights[3 * ci + 1], mu = class_weights[3 * ci + 2];
  const float omg = __fsub_rn(1.0f, gamma);
  const float needf = fmaxf((float)needd, 0.0f), fit_w = fmaxf(omg, 0.0f) * (1.0f + kSlack);
  const float widen = (needd < 0.0 && omg < 0.0f)
                          ? INFINITY
                          : kSlack * (fabsf(gamma) + fabsf(lambda) + fabsf(mu) + fabsf(omg));
  const int cs = ci * n_src + si, blocks4 = ((padded >> 6) + 3) & ~3;
  const float* gp_row = gp + (size_t)cs * padded;
  const float* pen_row = pen + (size_t)(ci * n_models + m) * padded;
  const float* b64 = bound + ((size_t)cs * n_models + m) * row;
  const float* b8 = b64 + blocks4;
  float known = -INFINITY;
  auto floor_key = [&]() { return fmaxf(-best.s[KT - 1], known) - widen; };
  for (int b = rest >> 3; __any(64 * b < mine); ++b) {
    if (parts > 1) {
      const uint32_t told = *static_cast<volatile uint32_t*>(floors);
      known = fmaxf(known, told ? key_float(told) : -INFINITY);
    }
    const float ub = fmaf(fit_w, needf * s_r64[b], b64[b]);
    const bool want64 = 64 * b < mine && !(ub < floor_key());
    if (!__any(want64)) continue;
    // the eight sub-blocks' bounds in two reads (one read of its own for each that a part takes):
    // these divergent reads are what a wavefront waits for
    float u8[8], r8[8];
    if (parts == 1) {
      load8(b8 + 8 * b, u8);
      load8(s_r8 + 8 * b, r8);
#pragma unroll
      for (int u = 0; u < 8; ++u) u8[u] = fmaf(fit_w, needf * r8[u], u8[u]);
    }
#pragma unroll 1
    for (int s = 8 * b + part; s < 8 * b + 8; s += parts) {
      if (!__any(8 * s < mine)) break;
      float us;
      if (parts == 1) {
        us = u8[0];
#pragma unroll
        for (int u = 0; u < 7; ++u) u8[u] = u8[u + 1];
      } else {
        us = fmaf(fit_w, needf * s_r8[s], b8[s]);
      }
      const bool want = s >= rest && want64 && 8 * s < mine && !(us < floor_key());
      if (!__any(want)) continue;
      float g[8], l[8];
      load8(gp_row + 8 * s, g);
      load8(pen_row + 8 * s, l);
      // the nodes whose plan may put them on the list, by the bound of a single node
      const ScalarSortedPlans sp = sorted_plans + 8 * s;
      const float reach = floor_key() + fminf(mu, 0.0f);
      uint32_t maybe = 0, nodes_any = 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const bool may = want && 8 * s + u < mine && !(need > sp[u].reach) &&
                         !(fmaf(fit_w, needf * sp[u].recip, g[u]) - fmaf(fmaxf(mu, 0.0f), sp[u].cost, l[u]) < reach);
        maybe |= may ? 1u << u : 0u;
        nodes_any |= __any(may) ? 1u << u : 0u;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        if (!((nodes_any >> u) & 1u)) continue;
        const int i = 8 * s + u;
        const float fit = __double2float_rn(__dmul_rn(needd, s_recip[i]));
        const float a = __fadd_rn(g[u], __fmul_rn(omg, fit));
        const int j = __builtin_amdgcn_readfirstlane((int)s_order[i]);
        // with mu >= 0 the fitness is at most the score with the plan's cheapest step
        const float most = -__fsub_rn(a, __fadd_rn(l[u], __fmul_rn(mu, sp[u].cost)));
        const bool go = ((maybe >> u) & 1u) &&
                        !(mu >= 0.0f && (most > best.s[KT - 1] || (most == best.s[KT - 1] && j > best.n[KT - 1])));
        if (!__any(go)) continue;
        float cost;
        if (plan_cost(plans + j, plan_steps, __dsub_rn(need, s_free[i]), go, cost) && go)
          best.push_lex(-__fsub_rn(a, __fadd_rn(l[u], __fmul_rn(mu, norm01(cost, lo_d, hi_d)))), j);
      }
      if (parts > 1 && best.s[KT - 1] < INFINITY) atomicMax(floors, float_key(-best.s[KT - 1]));
    }
  }
}

// Stages in turn, one per lane; the sorted node records, their original
// indices and the largest reciprocal of every block are staged in LDS once per workgroup. The best node
// alone fits 96 registers, five wavefronts a SIMD (one register more: 49.6 against 46.9 us on 719,712 stages).
enum : int { kNoPlans, kAlone, kShared };  // the last two with plans, kShared where several wavefronts take 64 stages
template <int KT, int kForm>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(KT == 1 && kForm == kNoPlans ? 5 : 4)))
void fitness_walk_kernel(const WalkArgs args) {
  constexpr bool kPlans = kForm != kNoPlans;
  const int32_t n_nodes = args.n_nodes, padded = args.padded, row = args.row, parts = args.parts;
  const SortedNode* __restrict__ nodes = args.nodes;
  const uint16_t* __restrict__ order = args.order;
  const float* __restrict__ bounds = args.bounds;
  RoundArgs in = round_args(&args);
  extern __shared__ __attribute__((aligned(16))) unsigned char s_raw[];
  const WalkLds lds = walk_lds(s_raw, padded);
  double *s_free = lds.free, *s_recip = lds.recip;
  float *s_r8 = lds.r8, *s_r64 = lds.r64;
  uint16_t* s_order = lds.order;
  const int blocks = padded >> 6, blocks4 = (blocks + 3) & ~3;
  const int tid = threadIdx.x, threads = blockDim.x;
  for (int i = tid; i < padded; i += threads) {
    const SortedNode nd = nodes[i];
    s_free[i] = nd.free;
    s_recip[i] = nd.recip;
    s_order[i] = order[i];
  }
  __syncthreads();
  // the largest reciprocal of a block, rounded up; padding counts as 0
  for (int b = tid; b < (padded >> 3); b += threads) {
    double r = 0.0;
    for (int u = 0; u < 8; ++u) r = fmax(r, s_recip[8 * b + u]);
    s_r8[b] = __double2float_ru(r);
  }
  __syncthreads();
  for (int b = tid; b < blocks4; b += threads) {
    float r = 0.0f;
    if (b < blocks)
      for (int u = 0; u < 8; ++u) r = fmaxf(r, s_r8[8 * b + u]);
    s_r64[b] = r;
  }
  __syncthreads();
  const float lo_d = bounds[4], hi_d = bounds[5];
  const float nd_fits = norm01(0.0f, lo_d, hi_d);   // normalised C_deg of a stage that fits

  // kShared: the first of `parts` wavefronts takes 64 stages, the others a part of the short pairs that it leaves
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int part = kForm == kShared ? wave & (parts - 1) : 0, group = kForm == kShared ? wave / parts : wave;
  const int per_block = kForm == kShared ? threads / parts : threads;
  const int64_t step = (int64_t)gridDim.x * per_block;
  const int64_t rounds = (args.n + step - 1) / step;   // workgroup-uniform: whole wavefronts vote below
  for (int64_t it = 0; it < rounds; ++it) {
    const int64_t stage = it * step + (int64_t)blockIdx.x * per_block + 64 * group + (tid & 63);
    ScalarPlans plans = nullptr;
    const maestro_plan_step* plan_steps = nullptr;
    if constexpr (kPlans) {
      const ColdArgs again = cold_args();
      in = round_args(again);
      plans = (ScalarPlans)again->plans;
      plan_steps = again->plan_steps;
    }
    const int32_t n_models = in.n_models, n_src = in.n_src;
    const float* class_weights = in.class_weights;
    TopK<KT> best;                                   // keys are -fitness: the smallest key is the best node
    best.init();
    bool ok = false;
    double need = NAN, needd = 0.0;
    float gamma = 0.0f, omg = 0.0f, lambda = 0.0f, mu = 0.0f;
    int cs = 0, cm = 0, m = 0;
    if (stage < in.n && part == 0) {
      const int32_t mi = in.model_id[stage], si = in.src_id[stage], ci = in.class_id[stage];
      ok = (uint32_t)mi < (uint32_t)n_models && (uint32_t)si < (uint32_t)n_src &&
           (uint32_t)ci < (uint32_t)in.n_classes;
      if (ok) {
        const double kv = in.kv_bytes[stage], rho = in.rho;
        need = (rho == 0.0) ? kv : __dmul_rn(kv, 1.0 + rho);
        needd = (double)__double2float_rn(need);
        gamma = class_weights[3 * ci];
        lambda = class_weights[3 * ci + 1];
        mu = class_weights[3 * ci + 2];
        omg = __fsub_rn(1.0f, gamma);
        cs = ci * n_src + si;
        cm = ci * n_models + mi;
        m = mi;
      }
    }
    const float* gp_row = in.gp + (size_t)cs * padded;
    const float* pen_row = in.pen + (size_t)cm * padded;
    const float* b64 = in.bound + ((size_t)cs * n_models + m) * row;
    const float* b8 = b64 + blocks4;
    const float* after = b8 + (padded >> 3);
    // bound of a block: fit_w * min(1, needf * largest reciprocal) + its table entry; a
    // negative demand with a negative fit weight has no such bound (every block is visited)
    const float needf = fmaxf((float)needd, 0.0f);
    const float fit_w = fmaxf(omg, 0.0f) * (1.0f + kSlack);
    const float widen = (needd < 0.0 && omg < 0.0f)
                            ? INFINITY
                            : kSlack * (fabsf(gamma) + fabsf(lambda) + fabsf(mu) + fabsf(omg));
    const float md = __fmul_rn(mu, nd_fits);
    // first sorted position that admits the stage
    int start = 0;
    if (ok) {
      int lo = 0, hi = n_nodes;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (need <= s_free[mid]) hi = mid;
        else lo = mid + 1;
      }
      start = lo;
    }
    // a lower bound of the k-th best fitness (the k-th best so far, or a bound from the tables), less the
    // widening of the bounds
    float known = -INFINITY;
    auto floor_key = [&]() { return fmaxf(-best.s[KT - 1], known) - widen; };

    // ---- the nodes that fall short, by their plans
    if constexpr (kPlans) {
      int mine = need == need ? start : 0;   // need is not a number: no score is
      int left = kForm == kShared ? kShortShared : kShortAlone, rest = -1;
      if (part == 0)
        for (int b = 0; rest < 0 && __any(64 * b < mine); ++b) {
          const float ub = fmaf(fit_w, needf * s_r64[b], b64[b]);
          const bool want64 = 64 * b < mine && !(ub < floor_key());
          if (!__any(want64)) continue;
          for (int s = 8 * b; s < 8 * b + 8; ++s) {
            if (!__any(8 * s < mine)) break;
            const float u8 = fmaf(fit_w, needf * s_r8[s], b8[s]);
            const bool want = want64 && 8 * s < mine && !(u8 < floor_key());
            if (!__any(want)) continue;
            if (left-- == 0) {
              rest = s;
              break;
            }
            float g[8], l[8];
            load8(gp_row + 8 * s, g);
            load8(pen_row + 8 * s, l);
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              const int i = 8 * s + u;
              const float fit = __double2float_rn(__dmul_rn(needd, s_recip[i]));
              const float a = __fadd_rn(g[u], __fmul_rn(omg, fit));
              // with mu >= 0 the fitness is at most the score with C_deg normalised to 0
              const bool go = want && i < mine && !(mu >= 0.0f && -__fsub_rn(a, l[u]) > best.s[KT - 1]);
              if (!__any(go)) continue;
              const int j = __builtin_amdgcn_readfirstlane((int)s_order[i]);
              float cost;
              if (plan_cost(plans + j, plan_steps, __dsub_rn(need, s_free[i]), go, cost) && go)
                best.push_lex(-__fsub_rn(a, __fadd_rn(l[u], __fmul_rn(mu, norm01(cost, lo_d, hi_d)))), j);
            }
          }
        }
      if constexpr (kForm == kShared) {
        uint32_t* floors = reinterpret_cast<uint32_t*>(s_raw + args.merge_at) + 64 * group + (tid & 63);
        // two sets in turn: a set is written again only behind the next stages' barrier
        int32_t* rests = reinterpret_cast<int32_t*>(s_raw + args.merge_at) + per_block + (it & 1) * kMaxGroups;
        float* m_key = reinterpret_cast<float*>(s_raw + args.merge_at) + per_block + 2 * kMaxGroups;
        int32_t* m_node = reinterpret_cast<int32_t*>(m_key + kSlots * KT * 64);
        uint16_t* mines = reinterpret_cast<uint16_t*>(m_node + kSlots * KT * 64) + 64 * group + (tid & 63);
        if (part == 0) {
          *floors = best.s[KT - 1] < INFINITY ? float_key(-best.s[KT - 1]) : 0u;
          *mines = (uint16_t)mine;
          rests[group] = rest;
        }
        __syncthreads();
        bool any = false;                // workgroup-uniform
        for (int g = 0; g * parts < (threads >> 6); ++g) any |= rests[g] >= 0;
        if (any) {
          rest = rests[group];
          mine = *mines;
          if (rest >= 0)
            short_pass<KT>(best, stage, mine, rest, part, parts, floors, s_raw);
          // the parts' lists meet in the first one's wavefront
          for (int g0 = 0; g0 * parts < (threads >> 6); g0 += kSlots)
            for (int p = 1; p < parts; ++p) {
              const bool slot = group >= g0 && group < g0 + kSlots;
              const int at = (group - g0) * KT * 64 + (tid & 63);
              if (slot && part == p)
#pragma unroll
                for (int i = 0; i < KT; ++i) {
                  m_key[at + 64 * i] = best.s[i];
                  m_node[at + 64 * i] = best.n[i];
                }
              __syncthreads();
              if (slot && part == 0)
#pragma unroll
                for (int i = 0; i < KT; ++i) best.push_lex(m_key[at + 64 * i], m_node[at + 64 * i]);
              __syncthreads();
            }
        }
      } else if (rest >= 0) {
        short_pass<KT>(best, stage, mine, rest, 0, 1, nullptr, s_raw);
      }
    }

    // A pair that fits and scores -inf (a penalty past the float32 range) takes no place in a list, nor
    // one held by a short pair of that score: such places count as held by a node below every other.
#pragma unroll
    for (int i = 0; i < KT; ++i)
      if (best.s[i] == INFINITY) best.n[i] ^= (int32_t)0x80000000;

    // ---- the nodes that admit the stage: those from `start` on
    const bool live = ok && start < n_nodes && need == need;
    const uint32_t room = (uint32_t)(n_nodes - start);
    auto score8 = [&](int sub) {
      float g[8], l[8];
      double r[8];
      load8(gp_row + 8 * sub, g);
      load8(pen_row + 8 * sub, l);
      const uint4 o = *reinterpret_cast<const uint4*>(s_order + 8 * sub);
      const uint32_t ow[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
      for (int u = 0; u < 8; u += 2) {
        const double2 d = *reinterpret_cast<const double2*>(s_recip + 8 * sub + u);
        r[u] = d.x;
        r[u + 1] = d.y;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float fit = __double2float_rn(__dmul_rn(needd, r[u]));
        const float a = __fadd_rn(g[u], __fmul_rn(omg, fit));
        const float p = kPlans ? __fadd_rn(l[u], md) : l[u];
        if ((uint32_t)(8 * sub + u - start) < room)
          best.push_lex(-__fsub_rn(a, p), (int32_t)((ow[u >> 1] >> (16 * (u & 1))) & 0xFFFFu));
      }
    };
    // The nodes that just fit come first, since the fit falls from there on: the sub-block where they
    // begin (and, for a list, the next one) gives a k-th best score that ends the pass over the bounds early.
    int seen = start >> 3;                                  // sub-blocks before it are done
    const bool ends_early = early_end(padded);
    if (live && ends_early) {
      score8(seen++);
      if (KT > 1 && 8 * seen < padded) score8(seen++);
    }
    // bounds of the eight sub-blocks of a block; those before `seen` are done
    auto sub_bounds = [&](int blk, float (&ub)[8]) {
      float t[8], r[8];
      load8(b8 + 8 * blk, t);
      load8(s_r8 + 8 * blk, r);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        ub[u] = 8 * blk + u < seen ? -INFINITY : fmaf(fit_w, fminf(needf * r[u], 1.0f), t[u]);
    };
    // Nodes that tie (idle nodes of one kind, a few distinct round-trip times) put every block's bound
    // within the widening of the k-th best score: a stage that meets several such bounds leaves the rest
    // to tie_pass.
    int ties = 0;
    auto tied = [&](float ub) { return (ties += ub <= widen - best.s[KT - 1] ? 1 : 0) > kTies; };
    // One pass over the bounds of the 64-node blocks from the stage's first one on: the two blocks
    // of the best bounds, the third best bound, and a lower bound of the k-th best fitness -- past
    // the first block every node admits the stage, so the node that holds a block's table entry
    // scores at least that entry plus the smallest fit term less the most that its C_deg term adds.
    // The pass ends where the largest table entry of all further blocks, with the fit term of the
    // next one (the largest of theirs), is below the k-th best score.
    const int blk0 = start >> 6;
    float top = -INFINITY, second = -INFINITY, third = -INFINITY;
    int arg = 0, arg2 = 0, end = blk0;
    if (live) {
      const float reach = floor_key();
      float low[KT];
#pragma unroll
      for (int i = 0; i < KT; ++i) low[i] = -INFINITY;
      int q = blk0 & ~3;
      do {
        const float4 t = *reinterpret_cast<const float4*>(b64 + q);
        const float4 r = *reinterpret_cast<const float4*>(s_r64 + q);
        const float tv[4] = {t.x, t.y, t.z, t.w}, rv[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int blk = q + u;
          const float ub =
              blk < blk0 || blk >= blocks ? -INFINITY : fmaf(fit_w, fminf(needf * rv[u], 1.0f), tv[u]);
          third = fmaxf(third, fminf(ub, second));
          arg2 = ub > top ? arg : ub > second ? blk : arg2;
          second = fmaxf(second, fminf(ub, top));
          arg = ub > top ? blk : arg;
          top = fmaxf(top, ub);
          float lb = blk > blk0 && blk < blocks ? tv[u] : -INFINITY;
#pragma unroll
          for (int i = 0; i < KT; ++i) {
            const float hi = fmaxf(low[i], lb);
            lb = fminf(low[i], lb);
            low[i] = hi;
          }
        }
        q += 4;
      } while (q < blocks && !(ends_early && fmaf(fit_w, fminf(needf * s_r64[q], 1.0f), after[q]) < reach));
      end = min(q, blocks);
      if (needd >= 0.0) known = low[KT - 1] - (fmaxf(-omg, 0.0f) + (kPlans ? md - fminf(mu, 0.0f) : 0.0f));
    }
    // The sub-blocks of those two blocks in descending order of their bounds while those reach the
    // k-th best score, then those of every other block whose bound still does.
    float ub[8], ub2[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) ub[u] = ub2[u] = -INFINITY;
    if (live && !(top < floor_key())) sub_bounds(arg, ub);
    if (live && second > -INFINITY && !(second < floor_key())) sub_bounds(arg2, ub2);
    for (;;) {
      int bs = 0;
      float bt = ub[0];
#pragma unroll
      for (int u = 1; u < 16; ++u) {
        const float v = u < 8 ? ub[u & 7] : ub2[u & 7];
        bs = v > bt ? u : bs;
        bt = fmaxf(bt, v);
      }
      if (!(bt > -INFINITY) || bt < floor_key()) break;
      if (tied(bt)) break;
      score8(8 * (bs < 8 ? arg : arg2) + (bs & 7));
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        ub[u] = u == bs ? -INFINITY : ub[u];
        ub2[u] = u + 8 == bs ? -INFINITY : ub2[u];
      }
    }
    const bool more = ties <= kTies && third > -INFINITY && !(third < floor_key());
    if (__any(more)) {
      uint64_t rest = 0;
      auto bound64 = [&](int blk) { return fmaf(fit_w, fminf(needf * s_r64[blk], 1.0f), b64[blk]); };
      if (more) {
        const float reach = floor_key();
#pragma unroll 2
        for (int q = blk0 & ~3; q < end; q += 4) {
          const float4 t = *reinterpret_cast<const float4*>(b64 + q);
          const float4 r = *reinterpret_cast<const float4*>(s_r64 + q);
          const float tv[4] = {t.x, t.y, t.z, t.w}, rv[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int blk = q + u;
            const bool in = blk >= blk0 && blk < end && blk != arg && blk != arg2;
            if (in && !(fmaf(fit_w, fminf(needf * rv[u], 1.0f), tv[u]) < reach)) rest |= 1ull << blk;
          }
        }
      }
      // taking the next block and scoring a sub-block are two steps of one loop, so that lanes at
      // different points of their lists share its iterations
      int blk = 0;
#pragma unroll
      for (int u = 0; u < 8; ++u) ub[u] = -INFINITY;
      for (;;) {
        int bs = 0;
        float bt = ub[0];
#pragma unroll
        for (int u = 1; u < 8; ++u) {
          bs = ub[u] > bt ? u : bs;
          bt = fmaxf(bt, ub[u]);
        }
        if (bt > -INFINITY && !(bt < floor_key())) {
          if (tied(bt)) break;
          score8(8 * blk + bs);
#pragma unroll
          for (int u = 0; u < 8; ++u) ub[u] = u == bs ? -INFINITY : ub[u];
        } else {
          do {   // the next block whose bound reaches the score as it now stands
            blk = __ffsll((unsigned long long)rest) - 1;
            rest &= rest - 1;
          } while (blk >= 0 && bound64(blk) < floor_key());
          if (blk < 0) break;
          sub_bounds(blk, ub);
        }
      }
    }

    if (ties > kTies) tie_pass<KT, kPlans>(best, stage, start, s_raw);

    if constexpr (kPlans) in = round_args(cold_args());
    if (stage < in.n && part == 0) {
#pragma unroll
      for (int i = 0; i < KT; ++i) {
        if (i < in.k) {
          const int32_t node = best.n[i] < 0 ? best.n[i] ^ (int32_t)0x80000000 : best.n[i];
          const bool some = node != kNoNode;
          in.node_idx[stage * in.k + i] = some ? node : -1;
          in.fitness[stage * in.k + i] = some ? -best.s[i] : -INFINITY;
        }
      }
    }
  }
}

constexpr size_t walk_lds_bytes(int32_t padded) {
  return (size_t)padded * (2 * sizeof(double) + sizeof(uint16_t)) + (size_t)(padded / 8) * sizeof(float) +
         (size_t)(((padded >> 6) + 3) & ~3) * sizeof(float);
}
// beside it where wavefronts share: floors and counts of short nodes, the resume points, the lists that meet
constexpr size_t share_lds_bytes(int kt, int threads, int parts) {
  return threads / parts * (sizeof(uint32_t) + sizeof(uint16_t)) + 2 * kMaxGroups * sizeof(int32_t) +
         kSlots * kt * 64 * (sizeof(float) + sizeof(int32_t));
}
// two workgroups a CU (one: 53 against 38 us for 131,072 stages)
static_assert(((walk_lds_bytes(kMaxNodes) + 15) & ~(size_t)15) + share_lds_bytes(4, kThreads, 2) <= 160 * 1024 / 2, "LDS");

}  // namespace

// Where the tables pay: from so many nodes on, from 2^pairs (stage, node) pairs on. Scoring every pair
// takes a latency that grows with the nodes a lane walks (17 us at 512 nodes, 45 at 2,000) plus about 1 us
// per 2^21 pairs; the tables and the walk take 22 to 60 us plus a time per stage that hardly grows with
// the nodes, but with the list: more blocks reach the fourth best score. So the lines lie higher for
// longer lists, and few nodes never pay. Where they lie was measured over three headroom
// distributions (0 .. 30 GB, 0 .. 288 GB, two modes) at 64 .. 4,096 nodes and 2^18 .. 2^28 pairs. Time of the
// tables over that of every pair, best .. worst distribution, below and at a line:
//   no plans  k = 1  128 nodes 1.09-1.21 at 2^25, 0.99-1.01 at 2^26; 256 1.11-1.21 at 2^24, 0.79-0.82 at 2^25;
//                    1,000 0.8-1.0 at 2^18 .. 2^23; 2,000 0.5-0.7 from 2^18 on; 96 nodes 1.06-1.09 at most
//             k = 2  128 nodes 0.99-1.19 at 2^28; 192 1.03-1.13 at 2^26, 0.94-0.99 at 2^27; 4,096 0.3-0.5
//             k = 4  384 nodes 0.81-1.14 at 2^28; 512 0.84-0.91 at 2^27; 4,096 0.5-0.7
//   plans     k = 1  128 nodes 0.78-1.13 at 2^25, 0.78-0.94 at 2^26; 192 1.06-1.16 at 2^24, 0.68-0.94 at 2^25;
//                    512 0.97-1.18 at 2^23, 0.84-0.99 at 2^24; 1,100 0.6-0.9; 96 nodes 0.99-1.06 at most
//             k = 2  128 nodes 0.79-1.05 at 2^28; 192 0.74-1.08 at 2^25, 0.71-0.92 at 2^26; 384 0.88-1.11 at 2^24,
//                    0.71-0.86 at 2^25; 700 0.9-1.0 at 2^24; 1,100 0.6-1.04
//             k = 4  256 nodes 0.70-1.17 at 2^28; 384 0.87-1.16 at 2^25, 0.64-1.02 at 2^26; 700 0.7-1.2 at 2^24,
//                    0.59-0.97 at 2^25; 1,100 0.7-1.4 up to 2^23, 0.56-0.95 at 2^25; 2,000 0.4-0.9
static bool tables_pay(int64_t n, int32_t n_nodes, int32_t k, bool plans) {
  struct Line {
    int32_t nodes;
    int pairs_log2;                      // 0: any batch
  };
  static constexpr Line kLines[2][3][4] = {
      {{{2048, 0}, {256, 25}, {128, 26}}, {{3072, 0}, {192, 27}}, {{3072, 0}, {512, 27}}},
      {{{1024, 0}, {512, 24}, {192, 25}, {128, 26}}, {{1024, 0}, {640, 24}, {384, 25}, {192, 26}},
       {{2000, 0}, {640, 25}, {384, 26}}}};
  for (const Line& line : kLines[plans][min(k, 3) - 1])
    if (line.nodes > 0 && n_nodes >= line.nodes && n * n_nodes >= (int64_t)1 << line.pairs_log2) return true;
  return false;
}

// The batches that the entry point takes. Its lines lie below those of tables_pay, between the two it
// scores every pair: a caller with a workspace need not know which of the two is faster. Many (class,
// source, model) combinations make the tables themselves the cost: 640 of them take 5 us at 4,096 nodes.
size_t fitness_workspace_bytes(int64_t n, int32_t n_models, int32_t n_nodes, int32_t n_src, int32_t n_classes,
                               int32_t k, bool plans) {
  if (k > 4 || n_nodes > kMaxNodes || n_nodes < 64) return 0;
  const int32_t always = plans ? 1024 : k == 1 ? 2048 : 3072;
  const int pairs_log2 = plans ? 24 : k == 1 ? 25 : 27;
  if (n_nodes < always && n * n_nodes < (int64_t)1 << pairs_log2) return 0;
  if ((int64_t)n_classes * n_src * n_models > 1024 + n / 8) return 0;
  return tables_of(n_models, n_nodes, n_src, n_classes).total;
}

maestro_status launch_route_fitness_pruned(int64_t n, const int32_t* model_id, const int32_t* src_id,
                                           const int32_t* class_id, const double* kv_bytes, int32_t n_models,
                                           int32_t n_nodes, int32_t n_src, int32_t n_classes, const double* free_bytes,
                                           const float* queue_ms, const float* act_ms, const uint64_t* resident_mask,
                                           const float* act_matrix, const float* deg_ms, const maestro_deg_plan* plans,
                                           const maestro_plan_step* plan_steps, const float* rtt_ms,
                                           const float* class_weights, const float* bounds, double rho, int32_t k,
                                           int32_t* node_idx, float* fitness, void* workspace, hipStream_t stream) {
  if (n == 0) return MAESTRO_OK;
  if (!tables_pay(n, n_nodes, k, plans != nullptr))
    return launch_route_fitness(n, model_id, src_id, class_id, kv_bytes, n_models, n_nodes, n_src, n_classes, free_bytes,
                                queue_ms, act_ms, resident_mask, act_matrix, deg_ms, plans, plan_steps, rtt_ms,
                                class_weights, bounds, rho, k, node_idx, fitness, stream);
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    return MAESTRO_ERR_LAUNCH;
  const Tables t = tables_of(n_models, n_nodes, n_src, n_classes);
  unsigned char* ws = static_cast<unsigned char*>(workspace);
  SortedNode* nodes = reinterpret_cast<SortedNode*>(ws + t.nodes);
  SortedPlan* sorted_plans = reinterpret_cast<SortedPlan*>(ws + t.plans);
  uint16_t* order = reinterpret_cast<uint16_t*>(ws + t.order);
  float* gp = reinterpret_cast<float*>(ws + t.gp);
  float* pen = reinterpret_cast<float*>(ws + t.pen);
  float* bound = reinterpret_cast<float*>(ws + t.bound);
  float* tr = reinterpret_cast<float*>(ws + t.tr);
  float* prox = reinterpret_cast<float*>(ws + t.prox);
  float* nd = reinterpret_cast<float*>(ws + t.nd);
  float* gp_top = reinterpret_cast<float*>(ws + t.gp_top);
  float* pen_low = reinterpret_cast<float*>(ws + t.pen_low);
  uint16_t* lowest = reinterpret_cast<uint16_t*>(ws + t.lowest);
  fitness_rank_kernel<<<dim3((unsigned)((t.padded + 15) / 16)), dim3(kRankThreads), 0, stream>>>(
      n_nodes, t.padded, n_models, n_src, free_bytes, queue_ms, act_ms, resident_mask, act_matrix,
      plans ? nullptr : deg_ms, rtt_ms, bounds, nodes, order, tr, prox, nd);
  const dim3 tgrid((unsigned)n_models, (unsigned)(n_classes + (plans ? kPlanRows : 0)),
                   (unsigned)(t.padded > 512 ? n_src : 1));
  const dim3 tblock((unsigned)(t.padded / 8));
  auto tables = plans ? fitness_tables_kernel<true> : fitness_tables_kernel<false>;
  tables<<<tgrid, tblock, 0, stream>>>(n_models, n_nodes, n_src, t.padded, t.row, tr, prox, nd, class_weights, order, gp,
                                       pen, bound, t.ends, gp_top, pen_low, lowest, nodes, plans, plan_steps, bounds,
                                       sorted_plans);
  const FitnessGrid shape = fitness_grid(n, t.padded, plans != nullptr, cus);
  const dim3 grid((unsigned)shape.blocks);
  const int threads = shape.threads;
#define MAESTRO_FITW(KT, FORM)                                                                                          \
  do {                                                                                                                \
    const size_t staged = (walk_lds_bytes(t.padded) + 15) & ~(size_t)15;                                              \
    const size_t lds = staged + (shape.parts > 1 ? share_lds_bytes(KT, threads, shape.parts) : 0);                    \
    if (lds > 65536 && hipFuncSetAttribute(reinterpret_cast<const void*>(&fitness_walk_kernel<KT, FORM>),               \
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)       \
      return MAESTRO_ERR_LAUNCH;                                                                                      \
    fitness_walk_kernel<KT, FORM><<<grid, dim3(threads), lds, stream>>>(                                               \
        WalkArgs{n, model_id, src_id, class_id, kv_bytes, n_models, n_nodes, n_src, n_classes, t.padded, t.row, nodes, \
                 order, gp, pen, bound, t.ends, gp_top, pen_low, lowest, sorted_plans, plans, plan_steps,             \
                 class_weights, bounds, rho, k, shape.parts, (int)staged, node_idx, fitness});                       \
  } while (0)
#define MAESTRO_FITW_KT(KT)                                \
  do {                                                     \
    if (!plans) MAESTRO_FITW(KT, kNoPlans);                \
    else if (shape.parts == 1) MAESTRO_FITW(KT, kAlone);   \
    else MAESTRO_FITW(KT, kShared);                        \
  } while (0)
  if (k == 1) MAESTRO_FITW_KT(1);
  else if (k == 2) MAESTRO_FITW_KT(2);
  else MAESTRO_FITW_KT(4);
#undef MAESTRO_FITW_KT
#undef MAESTRO_FITW
  return launch_status();
}

}  // namespace maestro
