// GPU executor: uploads a plan's step descriptors and operator blocks into the caller's
// workspace, walks the depth-first tree of sliced Kraus sites (every prefix computed once and
// kept in its level buffer), launches the steps (one each, or several as a chain, a block or a grid
// run), reduces each component's output in FP64 and assembles F_J on the device.  Also here: the
// batched submission (one persistent launch for the small components, hipGraph capture, lanes), the
// kernel autotuner, per-launch profiling, the early Definition 1 decision, and the FP32 rounding
// of operator blocks.
//
// Workspace layout (every region 256-byte aligned):
//   [descriptors][grid-run tables and flags][operator pools][constants][persistent tables]
//   [component outputs][sums][level buffers][level buffers of further lanes]
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cfloat>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "jf_internal.h"
#include "kernels.h"

namespace jf {

static_assert(LDS_RESIDENT_MAX == LDS_RESIDENT_LOG2, "the planner's LDS-resident components fit the persistent kernel");
static_assert(GRID_MAX_STEPS == GRID_STEPS && GRID_DIGITS == 5 && GRID_LOCAL == 10 && GRID_TILE == 11,
              "the planner's grid runs fit k_grid");
static_assert(BLOCK_MAX_STEPS == BLOCK_STEPS && BLOCK_STEPS <= CHAIN_STEPS, "the planner's blocks fit k_block");

namespace {

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

struct DevLayout {
  size_t desc_off = 0, pool_off = 0, const_off = 0, buf_off = 0, out_off = 0, sums_off = 0, total = 0;
  size_t image_end = 0;  // end of the host image (descriptors, operators, constants, LDS tables)
  size_t sumsq_off = 0;  // scratch of the two-pass sum of |t|^2 (2 SUMSQ_BLOCKS doubles)
  size_t res_off = 0;    // F_J, 1 - F_J, |Im|, written by the device; behind the failure word
  size_t lds_items_off = 0, lds_steps_off = 0;
  size_t ctr_off = 0;    // counter of the persistent launch's fused assembly (zero in the image)
  size_t fail_off = 0;   // failure word of the grid runs (zero in the image)
  size_t flags_off = 0;  // barrier flags of the grid runs (as in the image before a run that gives up)
  // the variants of a sliced component's first sliced level run in slice_lanes lanes: the level
  // buffers of the lanes after the first, lane_stride apart, lie behind total
  int slice_lanes = 1;
  size_t lane_off = 0, lane_stride = 0, lanes_total = 0;
  size_t grid_bytes = 0; // bytes of the workspace that only the grid runs and the blocks use
  bool grid = false;     // some run has a table
  std::vector<size_t> leaf_off;                           // per component with sliced wires: its leaf buffer
  std::vector<int> lds_comps;                             // components run by the persistent kernel
  int lds_steps = 0;
  std::vector<std::vector<size_t>> step_desc;             // per component, per step: descriptor offset
  std::vector<std::vector<size_t>> chain_desc;            // per component, per chain: descriptor offset
  std::vector<std::vector<size_t>> block_desc;            // per component, per block
  std::vector<std::vector<size_t>> run_desc;              // per component, per grid run: its steps' GridSteps,
                                                          // or kNoTable
  std::vector<std::vector<std::vector<size_t>>> step_b;   // per component, step, variant: B offset
  std::vector<std::vector<size_t>> level_buf;             // per component: 2 buffers per level, offsets in
                                                          // the buffer region [buf_off, total)
};

constexpr int BATCH_LANES = 4;               // hardware queues of a process
constexpr size_t kLaneBytes = size_t(64) << 20;  // level buffers of a member that shares the device

// Where a pass leaves its result (four doubles): pinned host memory and its device address, or nowhere
// (the result is copied out of the workspace).
struct Landing {
  double* host = nullptr;
  double* dev = nullptr;
  Landing entry(int i) const { return {host + 4 * i, dev + 4 * i}; }
};

struct DevState {
  DevLayout lay;
  std::vector<unsigned char> host_image;  // descriptors + pools + constants, uploaded as one copy
  const void* uploaded_to = nullptr;
  size_t uploaded_bytes = 0;
  hipGraphExec_t graph[BATCH_LANES] = {};       // a captured batch, one graph per lane
  const void* graph_ws = nullptr;
  hipStream_t graph_stream = nullptr;
  std::vector<unsigned long long> graph_plans;  // uids of the batch the cached graph was captured for
  std::vector<unsigned> graph_gens;         // and the kernel-choice generation of each plan
  int graph_lanes = 0;                          // 0: none captured
  unsigned variant_gen = 0;                 // bumped whenever a step's kernel choice changes
  // single-plan runs: the step program captured once per (workspace, stream, kernel choice)
  hipGraphExec_t run_graph = nullptr;
  const void* run_graph_ws = nullptr;
  hipStream_t run_graph_stream = nullptr;
  unsigned run_graph_gen = 0;
  hipStream_t own_stream = nullptr;         // used when the caller passes the null stream
  // the persistent launch of the small components runs on this stream beside the other
  // components' steps (fork and join by events, also inside a captured graph)
  hipStream_t side_stream = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  // the members of a batch, or the slices of a plan, run in lanes beside each other: the streams of the lanes after the first,
  // and the events that start them (the first) and end them
  hipStream_t lane_stream[BATCH_LANES - 1] = {};
  hipEvent_t ev_lane[BATCH_LANES] = {};
  // per component, per chain: 1 = run its steps one launch each (the autotuner found the chain
  // slower, or a kernel variant was forced on every step)
  std::vector<std::vector<char>> chain_off;
  // per component, per grid run: 1 = run its steps launch by launch (the autotuner found the run
  // slower, or a kernel variant was forced)
  std::vector<std::vector<char>> run_off;
  std::vector<std::vector<char>> block_off;  // the same for blocks
  long long grid_wait = 200000000;          // longest wait of a grid barrier: 2 s of the 100 MHz wall clock
  // a barrier gave up (the device is held by others): launch by launch from then on, so that the wait
  // is lost once, until the caller sets the wait, restores the kernel choice or tunes again
  bool grid_gave_up = false;
  bool validated = false;                   // the program passed validate_program (plans are immutable)
  hipEvent_t ev_order = nullptr, ev0 = nullptr, ev1 = nullptr;
  int grid_launches = 0, grid_steps = 0, lanes = 1, reruns = 0, joint_timings = 0;  // (jf_last_pass)
  // pinned host landing area of the component sums (4 doubles each): a pageable destination
  // costs the runtime a staging copy on every call, which small programs feel
  double* pinned_sums = nullptr;
  // pinned host landing area of F_J, 1 - F_J, |Im| (4 doubles), written by the assembly kernel
  // itself: allocated before the first enqueue of the allocating entry points, so every program
  // enqueued or captured after that writes it
  Landing res;
  // the results of a batch (of which this is the first plan): one per entry, since a plan may stand in
  // it twice
  Landing batch_res;
  int batch_entries = 0;
  // pinned host landing area of per-tuple traces: behind the result in its page where they fit, else
  // its own, up to 2 kTermChunk of them in two halves (the events: a half has landed)
  double2* pinned_terms = nullptr;
  double2* pinned_terms_dev = nullptr;
  hipEvent_t ev_terms[2] = {nullptr, nullptr};
};

std::atomic<unsigned> g_variant_gen{1};

// The first level of a component that iterates variants (-1: none).
int first_sliced(const ComponentProgram& cp) {
  for (size_t lv = 0; lv < cp.levels.size(); ++lv)
    if (cp.levels[lv].nvar > 1) return int(lv);
  return -1;
}

// The lanes of a plan's slices: 1 where nothing is sliced, where leaves add into one output (sliced
// wires), where a lane's level buffers are large enough to fill the device, and in captured plans (a
// graph submits its branches one after another).
int slice_lanes_of(const Program& P) {
  if (P.opt.flags & JF_FLAG_GRAPH) return 1;
  int lanes = 1;
  for (const ComponentProgram& cp : P.comps) {
    if (cp.lds_resident) continue;
    size_t bytes = 0;
    for (const Level& lv : cp.levels) bytes += 2 * lv.buf_bytes;
    if (bytes > kLaneBytes) return 1;
    const int lv = first_sliced(cp);
    if (lv >= 0 && !cp.accumulate) lanes = std::max(lanes, std::min(BATCH_LANES, cp.levels[lv].nvar));
  }
  return lanes;
}

std::mutex g_upload_mu;
// Plans whose tables a workspace holds: start address -> (plan, bytes of the plan's whole region:
// tables, buffers, outputs and sums).  A run writes its whole region, so an upload forgets every
// entry whose region overlaps the new one (a batch member inside a larger plan's buffers, or a
// larger plan over the members of an earlier batch); live entries never overlap.
struct Upload {
  const void* plan;
  size_t bytes;
};
std::map<const void*, Upload> g_last_upload;

// Forget every upload whose region meets [lo, hi) (caller holds g_upload_mu).
void forget_uploads(uintptr_t lo, uintptr_t hi) {
  for (auto it = g_last_upload.begin(); it != g_last_upload.end();) {
    const auto a = reinterpret_cast<uintptr_t>(it->first);
    if (a < hi && lo < a + std::max<size_t>(it->second.bytes, 1)) it = g_last_upload.erase(it);
    else ++it;
  }
}

int mode_of(const Step& st) {
  if (st.compute == C_F64) return st.in_prec == P_C64 ? KM_F32_TO_F64 : KM_F64;
  if (st.compute == C_F32) return st.two_term ? KM_F32X2 : KM_F32;
  return st.two_term ? KM_SPLIT4 : KM_SPLIT;
}

// Nearest BF16 number (ties to even) of an FP32 value, as an FP32 value.
float bf16_rne(float x) {
  uint32_t u;
  std::memcpy(&u, &x, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);
  u &= 0xFFFF0000u;
  float r;
  std::memcpy(&r, &u, 4);
  return r;
}
// Exact three-way split of an FP32 value into BF16 numbers: x = p[0] + p[1] + p[2] (each remainder
// is exact in FP32, and the last has at most 8 significant bits left).
void split3(float x, float p[3]) {
  p[0] = bf16_rne(x);
  const float r1 = x - p[0];
  p[1] = bf16_rne(r1);
  p[2] = bf16_rne(r1 - p[1]);
}

void balanced_round(const std::vector<cd>& M, std::vector<float>& out);

// Split-form operator block (kernels.h): P pieces of float4 entries, then the BF16 fragments of the
// Gauss form (single-term blocks) and of the real embedding.  Offsets in 16-byte units.
struct SplitLayout {
  int P = 3;
  long long gauss = -1, embed = -1, total = 0;
};
SplitLayout split_layout(const Step& st) {
  SplitLayout l;
  l.P = st.two_term ? 4 : 3;
  const long long pieces = (long long)l.P << (st.kS + st.kN);
  long long off = pieces;
  if (!st.two_term) {
    l.gauss = off;
    off += 576LL * split_gauss_mb(st.kN) * split_gauss_kc(st.kS);
  }
  l.embed = off;
  off += 64LL * l.P * split_embed_mb(st.kN) * split_embed_kc(st.kS);
  l.total = off;
  return l;
}
uint32_t bf16_bits(float x) {  // x is a BF16 number
  uint32_t u;
  std::memcpy(&u, &x, 4);
  return u >> 16;
}
uint32_t bf16_pair(float lo, float hi) { return bf16_bits(lo) | (bf16_bits(hi) << 16); }

// Fill one split-form block at dst from the FP64 block M (K x Nn, row-major [s][n]).
void fill_split_block(const Step& st, const std::vector<cd>& M, unsigned char* dst) {
  const SplitLayout l = split_layout(st);
  const int K = 1 << st.kS, Nn = 1 << st.kN;
  const size_t nb = M.size();
  // pieces of the FP32 block (balanced rounding for single-term blocks, as the FP32 steps round),
  // and for two-term blocks a fourth piece: the BF16 residual of the FP64 block
  std::vector<float> bal;
  if (!st.two_term) balanced_round(M, bal);
  std::vector<float> pc(size_t(l.P) * nb * 4, 0.f);  // [q][i][Re, Im, Re + Im, 0]
  for (size_t i = 0; i < nb; ++i) {
    const double re64 = M[i].real(), im64 = M[i].imag();
    const float re = st.two_term ? float(re64) : bal[2 * i], im = st.two_term ? float(im64) : bal[2 * i + 1];
    float pr[3], pi[3], ps[3];
    split3(re, pr);
    split3(im, pi);
    split3(re + im, ps);
    for (int q = 0; q < 3; ++q) {
      pc[(q * nb + i) * 4 + 0] = pr[q];
      pc[(q * nb + i) * 4 + 1] = pi[q];
      pc[(q * nb + i) * 4 + 2] = ps[q];
    }
    if (l.P == 4) {
      pc[(3 * nb + i) * 4 + 0] = bf16_rne(float(re64 - double(re)));
      pc[(3 * nb + i) * 4 + 1] = bf16_rne(float(im64 - double(im)));
    }
  }
  std::memcpy(dst, pc.data(), pc.size() * 4);
  auto piece = [&](int q, int s, int n, int x) {
    return (s < K && n < Nn) ? pc[((size_t(q) * nb) + size_t(s) * Nn + n) * 4 + x] : 0.f;
  };
  uint32_t* w = reinterpret_cast<uint32_t*>(dst);
  if (l.gauss >= 0) {
    const int MB = split_gauss_mb(st.kN), KC = split_gauss_kc(st.kS);
    for (int e = 0; e < 3 * MB * KC * 64 * 3; ++e) {
      const int q = e % 3, rest = e / 3, lane = rest & 63, r2 = rest >> 6;
      const int kc = r2 % KC, r3 = r2 / KC, mb = r3 % MB, x = r3 / MB;
      const int n = 16 * mb + (lane & 15), s0 = 32 * kc + 8 * (lane >> 4);
      for (int dd = 0; dd < 4; ++dd)
        w[4 * (l.gauss + e) + dd] = bf16_pair(piece(q, s0 + 2 * dd, n, x), piece(q, s0 + 2 * dd + 1, n, x));
    }
  }
  const int MB = split_embed_mb(st.kN), KC = split_embed_kc(st.kS);
  for (int e = 0; e < MB * KC * 64 * l.P; ++e) {
    const int q = e % l.P, rest = e / l.P, lane = rest & 63, r2 = rest >> 6;
    const int kc = r2 % KC, mb = r2 / KC;
    const int n = 8 * mb + ((lane & 15) >> 1), b = lane & 1, s0 = 16 * kc + 4 * (lane >> 4);
    for (int dd = 0; dd < 4; ++dd) {
      const float re = piece(q, s0 + dd, n, 0), im = piece(q, s0 + dd, n, 1);
      w[4 * (l.embed + e) + dd] = b == 0 ? bf16_pair(re, -im) : bf16_pair(im, re);
    }
  }
}

// FP32 image of a complex FP64 operator block for single-term FP32 steps.  Every entry is one of
// its two FP32 neighbours; among those choices the rounding keeps Re<B, fl(B) - B> (summed over
// real and imaginary parts) near zero.  In a miter network the rest of the network around a block
// is close to the block's inverse, so that inner product is the first-order change the rounding
// makes to the traces.  Round-to-nearest alone biases it whenever many entries share a value
// (the 1/sqrt(2) of H and T rounds down by 1.7e-8 in FP32, so such blocks shrink every trace by
// the same factor, step after step).  Start from round-to-nearest, then move single entries to
// their other neighbour, largest effect first, while that brings the sum closer to zero.
void balanced_round(const std::vector<cd>& M, std::vector<float>& out) {
  const size_t n = 2 * M.size();
  out.resize(n);
  struct Flip {
    double dT;
    size_t k;
    float alt;
  };
  std::vector<Flip> flips;
  double T = 0;
  for (size_t i = 0; i < n; ++i) {
    const double x = (i & 1) ? M[i / 2].imag() : M[i / 2].real();
    const float f = float(x);
    out[i] = f;
    const double d = double(f) - x;
    T += x * d;
    if (d != 0) {
      const float alt = std::nextafter(f, d > 0 ? -INFINITY : INFINITY);
      flips.push_back({x * (double(alt) - x - d), i, alt});
    }
  }
  std::sort(flips.begin(), flips.end(), [](const Flip& a, const Flip& b) {
    return std::fabs(a.dT) != std::fabs(b.dT) ? std::fabs(a.dT) > std::fabs(b.dT) : a.k < b.k;
  });
  for (const Flip& f : flips)
    if (std::fabs(T + f.dT) < std::fabs(T)) {
      T += f.dT;
      out[f.k] = f.alt;
    }
}

// The most bytes of a workspace that grid runs and blocks may add (the no-allocation scratch holds them
// beside JF_NOALLOC_BYTES): the tables of 3600 small steps.  A plan with more keeps its blocks and its
// longest runs, and the other steps get a launch each.
constexpr size_t kGridTableBytes = 4 << 20;
constexpr size_t kNoTable = ~size_t(0);  // the run has no table: a launch per step
constexpr size_t kResBehindFail = 32;
// A second set of barrier flags lies one word behind the first; a pass whose wait is 0 uses it.  The last
// workgroup's flag starts so far back there that the others' wait for it cannot end.
constexpr unsigned kFlagBehind = 0xC0000000u;

// The device descriptors of a grid run: where each step's tensors are (a step whose tensors hold at
// most 2^GRID_LOCAL elements runs in every workgroup's LDS; the last step of a run that is not the
// component's last leaves its output in memory) and its addressing.
std::vector<GridStep> grid_descriptors(const ComponentProgram& cp, const GridRun& run) {
  std::vector<GridStep> out(size_t(run.last - run.first));
  bool in_lds = false;  // the previous step's output
  for (int s = run.first; s < run.last; ++s) {
    const Step& st = cp.steps[s];
    GridTables tb;
    grid_tables(st, tb);
    GridStep& d = out[size_t(s - run.first)];
    std::memset(&d, 0, sizeof(d));
    const bool local = st.rA <= GRID_LOCAL && st.rC <= GRID_LOCAL;
    GridShape g = {};
    g.kS = st.kS;
    g.kN = st.kN;
    g.F = tb.F;
    g.lr = tb.lr;
    g.in32 = st.in_prec == P_C64;
    g.out32 = st.out_prec == P_C64;
    g.mode = mode_of(st);
    g.final_step = st.final_step;
    g.src_lds = in_lds || local;
    g.dst_lds = local && (st.final_step || s + 1 < run.last);
    in_lds = g.dst_lds;
    d.shape = g.pack();
    for (size_t i = 0; i < st.offS_A.size(); ++i) d.offS[i] = unsigned(st.offS_A[i]);
    for (size_t i = 0; i < st.offN_C.size(); ++i) d.offN[i] = unsigned(st.offN_C[i]);
    for (int q = 0; q < 16 * GRID_DIGITS; ++q) {
      d.digA[q] = tb.digA[q / 16][q % 16];
      d.digC[q] = tb.digC[q / 16][q % 16];
    }
  }
  return out;
}

// The device descriptor of a block.
BlockDesc block_descriptor(const ComponentProgram& cp, const Block& b) {
  BlockTables tb;
  block_tables(cp, b, tb);
  const int entry = cp.steps[b.first].compute == C_F64 ? 16 : 8;
  auto local = [&](const std::vector<int>& bits, long long i) {
    int o = 0;
    for (size_t k = 0; k < bits.size(); ++k)
      if ((i >> k) & 1) o ^= bits[k];
    return (unsigned short)(o * entry);
  };
  auto place = [](const std::vector<int>& pos, long long i) {
    long long o = 0;
    for (size_t k = 0; k < pos.size(); ++k) o |= ((i >> k) & 1LL) << pos[k];
    return o;
  };
  BlockDesc d;
  std::memset(&d, 0, sizeof(d));
  d.nTiles = b.nTiles;
  d.nsteps = b.last - b.first;
  d.T = b.T;
  d.Tin = int(b.Pin.size());
  d.Tout = int(b.Pout.size());
  d.f64 = cp.steps[b.first].compute == C_F64;
  for (int i = 0; i < 48; ++i) {
    const long long l = (long long)(i & 15) << (4 * (i >> 4));  // digit i >> 4 of an element index
    d.gIn[i] = place(b.Pin, l);
    d.gOut[i] = place(b.Pout, l);
    d.lIn[i] = local(tb.lin, l);
    d.lOut[i] = local(tb.lout, l);
  }
  for (int k = 0; k < 16; ++k) {
    const long long l = (long long)k * BLOCK_NT;
    d.gInK[k] = place(b.Pin, l);
    d.gOutK[k] = place(b.Pout, l);
    d.lInK[k] = local(tb.lin, l);
    d.lOutK[k] = local(tb.lout, l);
  }
  for (int i = 0; i < DMAXHI / 4 * 16; ++i) {
    const long long t = (long long)(i & 15) << (4 * (i >> 4));
    d.hbA[i] = place(b.hiA, t);
    d.hbC[i] = place(b.hiC, t);
  }
  for (int j = 0; j < d.nsteps; ++j) {
    const Step& st = cp.steps[b.first + j];
    BlockStepDesc& s = d.st[j];
    s.kS = st.kS;
    s.kN = st.kN;
    s.F = int(tb.f[j].size());
    s.boff = d.ops;
    d.ops += std::max(1, (1 << st.kS) >> 2) * std::max(1, (1 << st.kN) >> 4) * 64;
    for (int i = 0; i < 64; ++i) {
      const int g = (i >> 2) & 3, r = i & 3;
      s.s[i] = local(tb.s[j], 4 * (i & 15) + (i >> 4));
      s.n[i] = local(tb.n[j], (i & 48) + (d.f64 ? 4 * r + g : 4 * g + r));
    }
    for (int i = 0; i < 48; ++i) s.f[i] = local(tb.f[j], (long long)(i & 15) << (4 * (i >> 4)));
  }
  return d;
}

void build_layout(const Program& P, DevState& S) {
  DevLayout& L = S.lay;
  size_t off = 0;
  L.desc_off = 0;
  L.step_desc.resize(P.comps.size());
  for (size_t c = 0; c < P.comps.size(); ++c)
    for (size_t s = 0; s < P.comps[c].steps.size(); ++s) {
      L.step_desc[c].push_back(off);
      off += align256(sizeof(StepDesc));
    }
  L.chain_desc.resize(P.comps.size());
  S.chain_off.resize(P.comps.size());
  for (size_t c = 0; c < P.comps.size(); ++c) {
    S.chain_off[c].assign(P.comps[c].chains.size(), 0);
    for (size_t q = 0; q < P.comps[c].chains.size(); ++q) {
      L.chain_desc[c].push_back(off);
      off += align256(sizeof(ChainDesc));
    }
  }
  L.pool_off = off;
  L.step_b.resize(P.comps.size());
  for (size_t c = 0; c < P.comps.size(); ++c) {
    L.step_b[c].resize(P.comps[c].steps.size());
    for (size_t s = 0; s < P.comps[c].steps.size(); ++s) {
      const Step& st = P.comps[c].steps[s];
      // FP64 steps: double2 blocks; FP32 steps: hi and lo float2 blocks (b = hi + lo to ~48 bits);
      // split steps: pieces and fragments (split_layout)
      const size_t e = st.compute == C_F64 ? 16 : st.two_term ? 16 : 8;
      for (auto& b : st.B) {
        L.step_b[c][s].push_back(off);
        off += align256(st.compute == C_SPLIT ? size_t(split_layout(st).total) * 16 : b.size() * e);
      }
    }
  }
  L.const_off = off;
  off += 256;  // double2 one at +0, float2 one at +16
  for (size_t c = 0; c < P.comps.size(); ++c)
    if (P.comps[c].lds_resident) {
      L.lds_comps.push_back(int(c));
      L.lds_steps += int(P.comps[c].steps.size());
    }
  L.lds_items_off = off;
  off += align256(L.lds_comps.size() * sizeof(LdsItem));
  L.lds_steps_off = off;
  off += align256(size_t(L.lds_steps) * sizeof(LdsStep));
  L.ctr_off = off;
  L.fail_off = off + 128;
  L.res_off = L.fail_off + kResBehindFail;  // one copy reads both
  off += 256;
  // blocks: descriptors; grid runs: barrier flags and descriptors, the longest runs first
  L.run_desc.resize(P.comps.size());
  S.run_off.resize(P.comps.size());
  L.block_desc.resize(P.comps.size());
  S.block_off.resize(P.comps.size());
  L.slice_lanes = slice_lanes_of(P);
  const size_t flag_bytes = size_t(L.slice_lanes) * GRID_WGS * GRID_FLAG_STRIDE * sizeof(unsigned);
  const size_t table_end = off + kGridTableBytes;
  const size_t table_first = off;
  std::vector<std::pair<int, std::pair<size_t, size_t>>> order;  // -length, component, run
  for (size_t c = 0; c < P.comps.size(); ++c) {
    const ComponentProgram& cp = P.comps[c];
    if (cp.lds_resident) continue;
    for (size_t q = 0; q < cp.blocks.size() && off + align256(sizeof(BlockDesc)) <= table_end; ++q) {
      L.block_desc[c].push_back(off);
      off += align256(sizeof(BlockDesc));
    }
    S.block_off[c].assign(L.block_desc[c].size(), 0);
    L.run_desc[c].assign(cp.runs.size(), kNoTable);
    S.run_off[c].assign(cp.runs.size(), 0);
    for (size_t q = 0; q < cp.runs.size(); ++q) order.push_back({cp.runs[q].first - cp.runs[q].last, {c, q}});
  }
  std::sort(order.begin(), order.end());
  if (!order.empty() && off + flag_bytes <= table_end) {
    L.flags_off = off;
    off += flag_bytes;
    for (const auto& o : order) {
      const size_t bytes = align256(size_t(-o.first) * sizeof(GridStep));
      if (off + bytes > table_end) break;
      L.run_desc[o.second.first][o.second.second] = off;
      off += bytes;
      L.grid = true;
    }
  }
  L.grid_bytes = off - table_first;
  L.image_end = off;
  L.out_off = off;
  long long outn = 0;
  for (auto& cp : P.comps) outn += cp.out_len;
  off += align256(size_t(outn) * 16);
  L.leaf_off.assign(P.comps.size(), 0);
  for (size_t c = 0; c < P.comps.size(); ++c)
    if (P.comps[c].accumulate) {
      L.leaf_off[c] = off;
      off += align256(size_t(P.comps[c].leaf_len) * 16);
    }
  L.sums_off = off;
  off += align256(P.comps.size() * 4 * sizeof(double));
  L.sumsq_off = off;
  off += align256(2 * SUMSQ_BLOCKS * sizeof(double));
  // the level buffers last: the members of a batch that run one after another share one buffer
  // region (jf_fidelity_batch)
  L.buf_off = off;
  size_t maxbuf = 0;
  L.level_buf.resize(P.comps.size());
  for (size_t c = 0; c < P.comps.size(); ++c) {
    size_t o = 0;
    if (P.comps[c].lds_resident) {
      L.level_buf[c].assign(2 * P.comps[c].levels.size(), 0);
      continue;
    }
    for (auto& lv : P.comps[c].levels) {
      L.level_buf[c].push_back(o);
      o += align256(lv.buf_bytes);
      L.level_buf[c].push_back(o);
      o += align256(lv.buf_bytes);
    }
    maxbuf = std::max(maxbuf, o);
  }
  L.total = off + maxbuf;
  L.lane_off = align256(L.total);
  L.lane_stride = align256(maxbuf);
  L.lanes_total = L.slice_lanes > 1 ? L.lane_off + size_t(L.slice_lanes - 1) * L.lane_stride : L.total;

  // host image of descriptors, pools and constants
  S.host_image.assign(L.image_end, 0);
  for (int l = 0; L.grid && l < L.slice_lanes; ++l)
    std::memcpy(&S.host_image[L.flags_off + (size_t((l + 1) * GRID_WGS - 1) * GRID_FLAG_STRIDE + 1) * sizeof(unsigned)],
                &kFlagBehind, sizeof(kFlagBehind));
  for (size_t c = 0; c < P.comps.size(); ++c)
    for (size_t s = 0; s < P.comps[c].steps.size(); ++s) {
      const Step& st = P.comps[c].steps[s];
      StepDesc d;
      std::memset(&d, 0, sizeof(d));
      for (size_t i = 0; i < st.offS_A.size(); ++i) d.offS_A[i] = st.offS_A[i];
      for (size_t i = 0; i < st.offR_A.size(); ++i) d.offR_A[i] = st.offR_A[i];
      for (size_t i = 0; i < st.offN_C.size(); ++i) d.offN_C[i] = st.offN_C[i];
      for (size_t i = 0; i < st.offR_C.size(); ++i) d.offR_C[i] = st.offR_C[i];
      for (size_t i = 0; i < st.hiA.size(); ++i) {
        d.hiA[i] = st.hiA[i];
        d.hiC[i] = st.hiC[i];
      }
      d.nHi = int(st.hiA.size());
      for (int q = 0; q < DMAXHI / 4 * 16; ++q) {
        const int c = q >> 4, m = q & 15;
        long long a = 0, o = 0;
        for (int b = 0; b < 4; ++b)
          if (((m >> b) & 1) && 4 * c + b < d.nHi) {
            a |= 1LL << st.hiA[4 * c + b];
            o |= 1LL << st.hiC[4 * c + b];
          }
        d.digA[q] = a;
        d.digC[q] = o;
      }
      d.kS = st.kS;
      d.kN = st.kN;
      d.L = st.L;
      d.nTiles = st.nTiles;
      d.mode = mode_of(st);
      d.frag_gauss = d.frag_embed = -1;
      if (st.compute == C_SPLIT) {
        const SplitLayout sl = split_layout(st);
        d.frag_gauss = int(sl.gauss);
        d.frag_embed = int(sl.embed);
      }
      std::memcpy(&S.host_image[L.step_desc[c][s]], &d, sizeof(d));
      for (size_t v = 0; v < st.B.size(); ++v) {
        unsigned char* dst = &S.host_image[L.step_b[c][s][v]];
        if (st.compute == C_F64) {
          for (size_t i = 0; i < st.B[v].size(); ++i) {
            double re = st.B[v][i].real(), im = st.B[v][i].imag();
            std::memcpy(dst + 16 * i, &re, 8);
            std::memcpy(dst + 16 * i + 8, &im, 8);
          }
        } else if (st.compute == C_SPLIT) {
          fill_split_block(st, st.B[v], dst);
        } else {
          const size_t nb = st.B[v].size();
          std::vector<float> bal;
          const bool single = !st.two_term;
          if (single) balanced_round(st.B[v], bal);
          for (size_t i = 0; i < nb; ++i) {
            float re = float(st.B[v][i].real()), im = float(st.B[v][i].imag());
            if (single) {
              re = bal[2 * i];
              im = bal[2 * i + 1];
            }
            std::memcpy(dst + 8 * i, &re, 4);
            std::memcpy(dst + 8 * i + 4, &im, 4);
            if (!single) {
              float rl = float(st.B[v][i].real() - double(re)), il = float(st.B[v][i].imag() - double(im));
              std::memcpy(dst + 8 * (nb + i), &rl, 4);
              std::memcpy(dst + 8 * (nb + i) + 4, &il, 4);
            }
          }
        }
      }
    }
  for (size_t c = 0; c < P.comps.size(); ++c)
    for (size_t q = 0; q < P.comps[c].chains.size(); ++q) {
      const Chain& ch = P.comps[c].chains[q];
      ChainTables tb;
      chain_tables(P.comps[c], ch, tb);
      ChainDesc d;
      std::memset(&d, 0, sizeof(d));
      for (int i = 0; i < 48; ++i) d.gDig[i] = tb.gDig[i / 16][i % 16];
      for (size_t i = 0; i < ch.hi.size(); ++i) d.hi[i] = ch.hi[i];
      d.nTiles = ch.nTiles;
      d.nsteps = ch.last - ch.first;
      d.T = ch.T;
      d.nHi = int(ch.hi.size());
      d.split = P.comps[c].steps[ch.first].compute == C_SPLIT ? 1 : 0;
      int boff = 0;
      for (int j = 0; j < d.nsteps; ++j) {
        const Step& st = P.comps[c].steps[ch.first + j];
        d.st[j].kS = st.kS;
        d.st[j].boff = boff;
        d.st[j].frag = d.split ? int(split_layout(st).gauss) : 0;
        d.st[j].two = st.two_term ? 1 : 0;
        boff += chain_step_ops(st.kS, d.split != 0, st.two_term);
        for (size_t i = 0; i < tb.sOff[j].size(); ++i) d.st[j].sOff[i] = tb.sOff[j][i];
        for (int i = 0; i < 48; ++i) d.st[j].fDig[i] = tb.fDig[j][i];
      }
      d.ops = boff;
      std::memcpy(&S.host_image[L.chain_desc[c][q]], &d, sizeof(d));
    }
  for (size_t c = 0; c < P.comps.size(); ++c)
    for (size_t q = 0; q < L.run_desc[c].size(); ++q) {
      if (L.run_desc[c][q] == kNoTable) continue;
      const std::vector<GridStep> d = grid_descriptors(P.comps[c], P.comps[c].runs[q]);
      std::memcpy(&S.host_image[L.run_desc[c][q]], d.data(), d.size() * sizeof(GridStep));
    }
  for (size_t c = 0; c < P.comps.size(); ++c)
    for (size_t q = 0; q < L.block_desc[c].size(); ++q) {
      const BlockDesc d = block_descriptor(P.comps[c], P.comps[c].blocks[q]);
      std::memcpy(&S.host_image[L.block_desc[c][q]], &d, sizeof(d));
    }
  double one = 1.0, zero = 0.0;
  float onef = 1.0f, zerof = 0.0f;
  std::memcpy(&S.host_image[L.const_off], &one, 8);
  std::memcpy(&S.host_image[L.const_off + 8], &zero, 8);
  std::memcpy(&S.host_image[L.const_off + 16], &onef, 4);
  std::memcpy(&S.host_image[L.const_off + 20], &zerof, 4);
}

// Persistent-kernel tables of a plan whose workspace starts at ws (absolute device pointers).
void fill_lds_tables(const Program& P, const DevLayout& L, unsigned char* ws, LdsItem* items, LdsStep* steps,
                     int step_base) {
  int si = 0;
  for (size_t q = 0; q < L.lds_comps.size(); ++q) {
    const int c = L.lds_comps[q];
    const ComponentProgram& cp = P.comps[c];
    LdsItem it;
    it.first = step_base + si;
    it.count = int(cp.steps.size());
    it.out = reinterpret_cast<double2*>(ws + L.out_off + size_t(cp.out_off) * 16);
    it.sums = reinterpret_cast<double*>(ws + L.sums_off) + 4 * c;
    it.out_len = cp.out_len;
    items[q] = it;
    for (size_t k = 0; k < cp.steps.size(); ++k) {
      LdsStep e;
      e.desc = reinterpret_cast<const StepDesc*>(ws + L.step_desc[c][k]);
      e.B = ws + L.step_b[c][k][0];
      e.mode = mode_of(cp.steps[k]);
      e.final_step = cp.steps[k].final_step ? 1 : 0;
      e.kS = cp.steps[k].kS;
      e.kN = cp.steps[k].kN;
      e.L = cp.steps[k].L;
      e.nHi = int(cp.steps[k].hiA.size());
      e.log2_out = e.nHi + e.L + e.kN;
      e.pad = 0;
      steps[si++] = e;
    }
  }
}

DevState& state_of(jf_plan* p) {
  if (!p->dev) {
    auto* s = new DevState;
    build_layout(p->prog, *s);
    p->dev = s;
  }
  return *static_cast<DevState*>(p->dev);
}

#define JF_HIP(call)                                                                   \
  do {                                                                                 \
    hipError_t e_ = (call);                                                            \
    if (e_ != hipSuccess) {                                                            \
      set_error(std::string(#call) + ": " + hipGetErrorString(e_));                    \
      return JF_E_HIP;                                                                 \
    }                                                                                  \
  } while (0)

struct Prof {
  std::vector<hipEvent_t> ev;  // pairs around every contraction-step launch (owned)
  std::vector<jf_step_profile> rec;  // one per launch, ms filled in after the run
  double bytes = 0, flops = 0;
  Prof() = default;
  Prof(const Prof&) = delete;
  Prof& operator=(const Prof&) = delete;
  ~Prof() {
    for (auto e : ev) (void)hipEventDestroy(e);
  }
};

// Two timing events, destroyed on every way out of the scope that made them.
struct EventPair {
  hipEvent_t a = nullptr, b = nullptr;
  ~EventPair() {
    if (a) hipEventDestroy(a);
    if (b) hipEventDestroy(b);
  }
};

// Autotuning state of one run: which steps have been timed already.
struct Tune {
  int reps = 3;
  std::vector<std::vector<char>> done;
};

// Process-wide cache of tuned choices, keyed by step shape.
std::mutex g_tune_mu;
std::map<std::vector<long long>, int> g_tune_cache;

// Time every variant that can run this step (on its real input and output buffers) and keep the
// fastest in the host descriptor.  In-place steps are re-applied to their own output: the data
// is garbage afterwards, which is why tuning runs are never used for results.
jf_status tune_step(StepDesc* hd, const StepDesc* dd, const void* A, void* C, const void* B, hipStream_t stream,
                    int reps, bool inplace) {
  const std::vector<long long> key = {hd->mode, hd->kS, hd->kN, hd->L, hd->nTiles, inplace ? 1 : 0};
  {
    std::lock_guard<std::mutex> g(g_tune_mu);
    auto it = g_tune_cache.find(key);
    if (it != g_tune_cache.end()) {
      hd->variant = it->second;
      return JF_OK;
    }
  }
  EventPair ev;
  JF_HIP(hipEventCreate(&ev.a));
  JF_HIP(hipEventCreate(&ev.b));
  hipEvent_t e0 = ev.a, e1 = ev.b;
  int best = KV_AUTO;
  float best_ms = FLT_MAX;
  for (int v = KV_AUTO + 1; v < KV_COUNT; ++v) {
    if (!variant_applies(*hd, v)) continue;
    hd->variant = v;
    JF_HIP(launch_step(dd, *hd, A, C, B, stream));  // warm-up
    JF_HIP(hipEventRecord(e0, stream));
    for (int r = 0; r < reps; ++r) JF_HIP(launch_step(dd, *hd, A, C, B, stream));
    JF_HIP(hipEventRecord(e1, stream));
    JF_HIP(hipEventSynchronize(e1));
    float ms = 0;
    JF_HIP(hipEventElapsedTime(&ms, e0, e1));
    if (ms < best_ms) {
      best_ms = ms;
      best = v;
    }
  }
  hd->variant = best;
  std::lock_guard<std::mutex> g(g_tune_mu);
  g_tune_cache[key] = best;
  return JF_OK;
}

// Process-wide cache of chain decisions (1 = run the steps one launch each), keyed by the chain's
// tile shape and its steps' shapes and kernels.
std::map<std::vector<long long>, int> g_chain_cache;

// Time a chain against its steps run one launch each (every step with its tuned kernel, in place
// on the chain's output after the first) and keep the faster.  Like tune_step, this clobbers the
// data.
jf_status tune_chain(DevState& S, size_t c, int q, const ChainDesc* dd, const ChainDesc& hd,
                     const void* A, void* C, const ChainOps& ops, const std::vector<const StepDesc*>& sdd,
                     const std::vector<const StepDesc*>& shd, hipStream_t stream, int reps) {
  std::vector<long long> key = {hd.T, hd.nTiles, A == C ? 1 : 0, hd.split};
  for (const StepDesc* h : shd) {
    key.push_back(h->kS);
    key.push_back(resolve_variant(*h));
  }
  {
    std::lock_guard<std::mutex> g(g_tune_mu);
    auto it = g_chain_cache.find(key);
    if (it != g_chain_cache.end()) {
      S.chain_off[c][q] = char(it->second);
      return JF_OK;
    }
  }
  auto run_steps = [&]() -> hipError_t {
    for (size_t j = 0; j < shd.size(); ++j) {
      const hipError_t e = launch_step(sdd[j], *shd[j], j == 0 ? A : C, C, ops.B[j], stream);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  };
  EventPair ev;
  JF_HIP(hipEventCreate(&ev.a));
  JF_HIP(hipEventCreate(&ev.b));
  hipEvent_t e0 = ev.a, e1 = ev.b;
  float ms[2] = {0, 0};
  for (int mode = 0; mode < 2; ++mode) {
    JF_HIP(mode == 0 ? launch_chain(dd, hd, A, C, ops, stream) : run_steps());  // warm-up
    JF_HIP(hipEventRecord(e0, stream));
    for (int r = 0; r < reps; ++r) JF_HIP(mode == 0 ? launch_chain(dd, hd, A, C, ops, stream) : run_steps());
    JF_HIP(hipEventRecord(e1, stream));
    JF_HIP(hipEventSynchronize(e1));
    JF_HIP(hipEventElapsedTime(&ms[mode], e0, e1));
  }
  S.chain_off[c][q] = ms[0] <= ms[1] ? 0 : 1;
  std::lock_guard<std::mutex> g(g_tune_mu);
  g_chain_cache[key] = S.chain_off[c][q];
  return JF_OK;
}

// How a pass uses grid runs, and what their last launch took over.
struct GridUse {
  bool assemble = false;   // nothing is left to do before the assembly once this component is summed
  bool summed = false;     // the component's sum of |t|^2 is done
  bool assembled = false;  // and the assembly
  double* host = nullptr;  // where the assembly leaves the result (Landing::dev)
  int lane = 0;            // runs beside each other have flags of their own
};

int run_starting_at(const ComponentProgram& cp, int si) {
  for (size_t q = 0; q < cp.runs.size(); ++q)
    if (cp.runs[q].first == si) return int(q);
  return -1;
}

// The block that runs from step si on, or -1; and whether such a block takes any step of a chain.
int block_starting_at(const ComponentProgram& cp, const DevState& S, const DevLayout& L, size_t c, int si) {
  for (size_t q = 0; q < L.block_desc[c].size(); ++q)
    if (cp.blocks[q].first == si && !S.block_off[c][q]) return int(q);
  return -1;
}
bool chain_taken(const ComponentProgram& cp, const DevState& S, const DevLayout& L, size_t c, const Chain& ch) {
  for (size_t q = 0; q < L.block_desc[c].size(); ++q)
    if (!S.block_off[c][q] && cp.blocks[q].first < ch.last && ch.first < cp.blocks[q].last) return true;
  return false;
}

// The buffer that holds a grid run's output: the steps that write memory alternate between the
// level's buffers as k_grid does.
const void* grid_output(const GridArgs& a) {
  const void* cur = a.in;
  for (int i = 0; i < a.n; ++i)
    if (!GridShape::unpack(a.shape[i]).dst_lds) cur = cur == a.buf[0] ? a.buf[1] : a.buf[0];
  return cur;
}

AssembleArgs assemble_args(jf_plan* p, unsigned char* ws, double* host);
jf_status enqueue_steps(jf_plan* p, unsigned char* ws, unsigned char* bufs, hipStream_t stream, size_t c, int lv,
                        int from, int to, const std::vector<int>& vv, const void* cur, long long base, const void** end,
                        Prof* prof, Tune* tune, GridUse* gu);

// Process-wide cache of the decisions on grid runs and blocks (1 = launch by launch), keyed by what
// either way runs: the steps' shapes, the chains they would run in, and a block's tile (its places in
// memory decide how much of a line a tile takes).
std::map<std::vector<long long>, int> g_run_cache;

// After a give-up: no grid runs from here on, in captured programs neither, and the failure word and
// the barrier flags as they were uploaded.
jf_status leave_grid(jf_plan* p, unsigned char* ws, hipStream_t stream) {
  DevState& S = state_of(p);
  const DevLayout& L = S.lay;
  S.grid_gave_up = true;
  S.variant_gen = g_variant_gen.fetch_add(1);
  JF_HIP(hipMemcpyAsync(ws + L.fail_off, &S.host_image[L.fail_off], sizeof(unsigned), hipMemcpyHostToDevice, stream));
  JF_HIP(hipMemcpyAsync(ws + L.flags_off, &S.host_image[L.flags_off],
                        size_t(L.slice_lanes) * GRID_WGS * GRID_FLAG_STRIDE * sizeof(unsigned), hipMemcpyHostToDevice,
                        stream));
  return JF_OK;
}

// Time steps [first, last) as one launch (a grid run, or the block blk, switched off by `off`) against their
// own launches (tuned, chains included) and keep the faster.  A grid run that gave up its barrier has
// no time (the launches after that do nothing): its steps get their own launches, for this plan alone.
jf_status tune_joint(jf_plan* p, unsigned char* ws, unsigned char* bufs, hipStream_t stream, size_t c, int lv, int first,
                     int last, char& off, const Block* blk, const std::vector<int>& vv, const void* in, long long base,
                     int reps) {
  const ComponentProgram& cp = p->prog.comps[c];
  DevState& S = state_of(p);
  std::vector<long long> key = {blk ? 1LL : 0LL};
  if (blk) {
    key.insert(key.end(), {(long long)blk->T, blk->nTiles, (long long)blk->Pin.size()});
    key.insert(key.end(), blk->Pin.begin(), blk->Pin.end());
    key.insert(key.end(), blk->Pout.begin(), blk->Pout.end());
  }
  for (int s = first; s < last; ++s) {
    const Step& st = cp.steps[s];
    for (long long v : {(long long)st.kS, (long long)st.kN, (long long)st.rA, (long long)st.rC, (long long)mode_of(st),
                        (long long)st.final_step})
      key.push_back(v);
    if (st.chain >= 0 && !S.chain_off[c][st.chain]) {  // relative extents, never 0 apart
      const Chain& ch = cp.chains[st.chain];
      key.insert(key.end(), {(long long)(ch.first - s), (long long)(ch.last - s)});
    } else {
      key.insert(key.end(), {0LL, 0LL});
    }
  }
  {
    std::lock_guard<std::mutex> g(g_tune_mu);
    auto it = g_run_cache.find(key);
    if (it != g_run_cache.end()) {
      off = char(it->second);
      return JF_OK;
    }
  }
  EventPair ev;
  JF_HIP(hipEventCreate(&ev.a));
  JF_HIP(hipEventCreate(&ev.b));
  float ms[2] = {0, 0};
  for (int mode = 0; mode < 2; ++mode) {
    off = char(mode);
    const void* end = nullptr;
    GridUse gu;
    for (int r = 0; r <= reps; ++r) {  // the first is the warm-up
      if (r == 1) JF_HIP(hipEventRecord(ev.a, stream));
      const jf_status st = enqueue_steps(p, ws, bufs, stream, c, lv, first, last, vv, in, base, &end, nullptr, nullptr,
                                         blk ? nullptr : &gu);
      if (st != JF_OK) return st;
    }
    JF_HIP(hipEventRecord(ev.b, stream));
    JF_HIP(hipEventSynchronize(ev.b));
    JF_HIP(hipEventElapsedTime(&ms[mode], ev.a, ev.b));
    if (mode == 0 && !blk) {
      unsigned failed = 0;
      JF_HIP(hipMemcpyAsync(&failed, ws + S.lay.fail_off, sizeof(failed), hipMemcpyDeviceToHost, stream));
      JF_HIP(hipStreamSynchronize(stream));
      if (failed) {
        off = 1;
        return leave_grid(p, ws, stream);
      }
    }
  }
  off = ms[0] <= ms[1] ? 0 : 1;
  ++S.joint_timings;
  std::lock_guard<std::mutex> g(g_tune_mu);
  g_run_cache[key] = off;
  return JF_OK;
}

// Enqueue steps [from, to) of level lv of component c (the levels at the values vv) on the tensor
// `cur`, the component's output at element offset `base`; *end receives the last output (no
// synchronisation).  gu not null: grid runs go out as one launch each.
jf_status enqueue_steps(jf_plan* p, unsigned char* ws, unsigned char* bufs, hipStream_t stream, size_t c, int lv,
                        int from, int to, const std::vector<int>& vv, const void* cur, long long base, const void** end,
                        Prof* prof, Tune* tune, GridUse* gu) {
  const ComponentProgram& cp = p->prog.comps[c];
  DevState& S = state_of(p);
  const DevLayout& L = S.lay;
  unsigned char* out = ws + L.out_off + size_t(cp.out_off) * 16;
  unsigned char* b0 = bufs + L.level_buf[c][2 * lv];
  unsigned char* b1 = bufs + L.level_buf[c][2 * lv + 1];
  for (int si = from; si < to; ++si) {
    const Step& st = cp.steps[si];
    if (gu) {
      const int q = run_starting_at(cp, si);
      if (q >= 0 && L.run_desc[c][q] != kNoTable && !S.run_off[c][q]) {
        const GridRun& run = cp.runs[q];
        GridArgs a = {};
        a.steps = reinterpret_cast<const GridStep*>(ws + L.run_desc[c][q]);
        a.n = run.last - run.first;
        a.in = cur;
        a.buf[0] = b0;
        a.buf[1] = b1;
        a.flags = reinterpret_cast<unsigned*>(ws + L.flags_off) + gu->lane * GRID_WGS * GRID_FLAG_STRIDE +
                  (S.grid_wait > 0 ? 0 : 1);
        a.fail = reinterpret_cast<unsigned*>(ws + L.fail_off);
        a.limit = S.grid_wait;
        const GridStep* hs = reinterpret_cast<const GridStep*>(&S.host_image[L.run_desc[c][q]]);
        for (int k = 0; k < a.n; ++k) a.shape[k] = hs[k].shape;
        for (int k = run.first; k < run.last; ++k)
          a.B[k - run.first] = ws + L.step_b[c][k][variant_index(cp, cp.steps[k], vv)];
        const Step& fs = cp.steps[run.last - 1];
        if (fs.final_step) {
          a.out = cp.accumulate ? static_cast<void*>(ws + L.leaf_off[c]) : static_cast<void*>(out + size_t(base) * 16);
          // one workgroup sums the output, so a large one keeps its own launches (as launch_sumsq)
          if (fs.rC <= 14 && cp.leaves == 1 && !cp.accumulate && cp.out_len == (1LL << fs.rC)) {
            a.sums = reinterpret_cast<double*>(ws + L.sums_off) + 4 * c;
            gu->summed = true;
            if (gu->assemble) {
              a.as = assemble_args(p, ws, gu->host);
              gu->assembled = true;
            }
          }
        }
        JF_HIP(launch_grid(a, stream));
        ++S.grid_launches;
        S.grid_steps += a.n;
        if (fs.final_step) {
          if (cp.accumulate) JF_HIP(launch_accumulate(out + size_t(base) * 16, a.out, cp.leaf_len, stream));
          cur = a.out;
        } else {
          cur = grid_output(a);
        }
        si = run.last - 1;
        continue;
      }
    }
    const int bq = tune ? -1 : block_starting_at(cp, S, L, c, si);
    if (bq >= 0) {
      // a block: steps [first, last) in one launch, from one level buffer to the other
      const Block& blk = cp.blocks[bq];
      void* dst = cur == b0 ? b1 : b0;
      ChainOps ops = {};
      for (int q = blk.first; q < blk.last; ++q)
        ops.B[q - blk.first] = ws + L.step_b[c][q][variant_index(cp, cp.steps[q], vv)];
      const BlockDesc* dd = reinterpret_cast<const BlockDesc*>(ws + L.block_desc[c][bq]);
      const BlockDesc& hd = *reinterpret_cast<const BlockDesc*>(&S.host_image[L.block_desc[c][bq]]);
      if (prof) {
        hipEvent_t a = nullptr, b = nullptr;
        JF_HIP(hipEventCreate(&a));
        prof->ev.push_back(a);
        JF_HIP(hipEventCreate(&b));
        prof->ev.push_back(b);
        set_launch_events(a, b);
        const hipError_t le = launch_block(dd, hd, cur, dst, ops, stream);
        set_launch_events(nullptr, nullptr);
        JF_HIP(le);
        prof->bytes += blk.bytes;
        prof->flops += blk.flops;
        jf_step_profile r = {};
        r.flops = blk.flops;
        r.bytes = blk.bytes;
        for (int j = 0; j < hd.nsteps; ++j) {
          r.kS = std::max(r.kS, hd.st[j].kS);
          r.kN = std::max(r.kN, hd.st[j].kN);
        }
        r.L = hd.T;
        r.mode = hd.f64 ? KM_F64 : KM_F32;
        r.variant = KV_BLOCK;
        r.component = int(c);
        r.steps = hd.nsteps;
        r.threads = BLOCK_NT;
        prof->rec.push_back(r);
      } else {
        JF_HIP(launch_block(dd, hd, cur, dst, ops, stream));
      }
      cur = dst;
      si = blk.last - 1;
      continue;
    }
    if (st.chain >= 0 && cp.chains[st.chain].first == si && (tune || !S.chain_off[c][st.chain]) &&
        (tune || !chain_taken(cp, S, L, c, cp.chains[st.chain]))) {
      // a chain: steps [first, last) in one launch, in place when the input is this level's
      const Chain& ch = cp.chains[st.chain];
      void* dst = (cur == b0 || cur == b1) ? const_cast<void*>(cur) : b0;
      ChainOps ops = {};
      std::vector<const StepDesc*> sdd, shd;
      for (int q = ch.first; q < ch.last; ++q) {
        ops.B[q - ch.first] = ws + L.step_b[c][q][variant_index(cp, cp.steps[q], vv)];
        sdd.push_back(reinterpret_cast<const StepDesc*>(ws + L.step_desc[c][q]));
        shd.push_back(reinterpret_cast<const StepDesc*>(&S.host_image[L.step_desc[c][q]]));
      }
      const ChainDesc* dd = reinterpret_cast<const ChainDesc*>(ws + L.chain_desc[c][st.chain]);
      const ChainDesc& hd = *reinterpret_cast<const ChainDesc*>(&S.host_image[L.chain_desc[c][st.chain]]);
      if (tune && !tune->done[c][si]) {
        for (int q = ch.first; q < ch.last; ++q) {  // the steps' own kernels first
          jf_status ts = tune_step(const_cast<StepDesc*>(shd[q - ch.first]), sdd[q - ch.first], q == ch.first ? cur : dst,
                                   dst, ops.B[q - ch.first], stream, tune->reps, q == ch.first ? dst == cur : true);
          if (ts != JF_OK) return ts;
          tune->done[c][q] = 1;
        }
        jf_status ts = tune_chain(S, c, st.chain, dd, hd, cur, dst, ops, sdd, shd, stream, tune->reps);
        if (ts != JF_OK) return ts;
      }
      if (!S.chain_off[c][st.chain]) {
        if (prof) {
          hipEvent_t a = nullptr, b = nullptr;
          JF_HIP(hipEventCreate(&a));
          prof->ev.push_back(a);
          JF_HIP(hipEventCreate(&b));
          prof->ev.push_back(b);
          set_launch_events(a, b);
          const hipError_t le = launch_chain(dd, hd, cur, dst, ops, stream);
          set_launch_events(nullptr, nullptr);
          JF_HIP(le);
          prof->bytes += ch.bytes;
          prof->flops += ch.flops;
          jf_step_profile r = {};
          r.flops = ch.flops;
          r.bytes = ch.bytes;
          for (const StepDesc* h : shd) r.kS = std::max(r.kS, h->kS);
          r.kN = r.kS;
          r.L = ch.T;
          bool pairs = false;
          for (int j = 0; j < hd.nsteps; ++j) pairs = pairs || hd.st[j].two;
          r.mode = hd.split ? KM_SPLIT : pairs ? KM_F32X2 : KM_F32;
          r.variant = KV_CHAIN;
          r.component = int(c);
          r.steps = ch.last - ch.first;
          r.threads = chain_threads(hd);
          prof->rec.push_back(r);
        } else {
          JF_HIP(launch_chain(dd, hd, cur, dst, ops, stream));
        }
        cur = dst;
        si = ch.last - 1;
        continue;
      }
    }
    void* dst;
    if (st.final_step) {
      // with sliced wires the leaf's partial result goes to the leaf buffer and is added in below
      dst = cp.accumulate ? static_cast<void*>(ws + L.leaf_off[c]) : static_cast<void*>(out + size_t(base) * 16);
    } else if (st.inplace_ok && st.in_prec == st.out_prec && (cur == b0 || cur == b1)) {
      dst = const_cast<void*>(cur);
    } else {
      dst = (cur == b0) ? b1 : b0;
    }
    const size_t var = variant_index(cp, st, vv);
    const StepDesc* dd = reinterpret_cast<const StepDesc*>(ws + L.step_desc[c][si]);
    const StepDesc* hd = reinterpret_cast<const StepDesc*>(&S.host_image[L.step_desc[c][si]]);
    const void* B = ws + L.step_b[c][si][var];
    if (tune && !tune->done[c][si]) {
      jf_status ts = tune_step(const_cast<StepDesc*>(hd), dd, cur, dst, B, stream, tune->reps, dst == cur);
      if (ts != JF_OK) return ts;
      tune->done[c][si] = 1;
    }
    if (prof) {
      hipEvent_t a = nullptr, b = nullptr;
      JF_HIP(hipEventCreate(&a));
      prof->ev.push_back(a);
      JF_HIP(hipEventCreate(&b));
      prof->ev.push_back(b);
      set_launch_events(a, b);
      const hipError_t le = launch_step(dd, *hd, cur, dst, B, stream);
      set_launch_events(nullptr, nullptr);
      JF_HIP(le);
      prof->bytes += st.bytes;
      prof->flops += st.flops;
      jf_step_profile r = {};
      r.flops = st.flops;
      r.bytes = st.bytes;
      r.kS = st.kS;
      r.kN = st.kN;
      r.L = st.L;
      r.mode = hd->mode;
      r.variant = resolve_variant(*hd);
      r.component = int(c);
      r.steps = 1;
      r.threads = step_threads(*hd);
      prof->rec.push_back(r);
    } else {
      JF_HIP(launch_step(dd, *hd, cur, dst, B, stream));
    }
    if (st.final_step && cp.accumulate)
      JF_HIP(launch_accumulate(out + size_t(base) * 16, dst, cp.leaf_len, stream));
    cur = dst;
  }
  *end = cur;
  return JF_OK;
}

// Enqueue the steps of level lv from `parent` (nullptr: the constant 1 of the first step's precision).
// On the first visit of a tuning pass the level's grid runs and blocks are timed too, after their steps.
jf_status enqueue_level(jf_plan* p, unsigned char* ws, unsigned char* bufs, hipStream_t stream, size_t c, int lv,
                        const std::vector<int>& vv, const void* parent, long long base, const void** end, Prof* prof,
                        Tune* tune, GridUse* gu) {
  const ComponentProgram& cp = p->prog.comps[c];
  DevState& S = state_of(p);
  const DevLayout& L = S.lay;
  const Level& lev = cp.levels[lv];
  const void* cur = parent;
  if (!cur) {
    const Step& s0 = cp.steps[lev.first < lev.last ? lev.first : 0];
    cur = ws + L.const_off + (s0.in_prec == P_C64 ? 16 : 0);
  }
  const void* start = cur;
  jf_status st = enqueue_steps(p, ws, bufs, stream, c, lv, lev.first, lev.last, vv, cur, base, end, prof, tune,
                               prof || tune ? nullptr : gu);
  if (st != JF_OK || !tune) return st;
  auto joint = [&](int first, int last, char& off, const Block* blk) {
    if (first < lev.first || last > lev.last || tune->done[c][first] == 2) return JF_OK;
    // the input: the level's, or what an earlier step of the level left in a level buffer (the data
    // is garbage by now, which the timing does not see)
    const void* in = first == lev.first ? start : bufs + L.level_buf[c][2 * lv + 1];
    tune->done[c][first] = 2;
    return tune_joint(p, ws, bufs, stream, c, lv, first, last, off, blk, vv, in, base, tune->reps);
  };
  for (size_t q = 0; q < L.run_desc[c].size() && gu && !S.grid_gave_up && st == JF_OK; ++q)
    if (L.run_desc[c][q] != kNoTable) st = joint(cp.runs[q].first, cp.runs[q].last, S.run_off[c][q], nullptr);
  for (size_t q = 0; q < L.block_desc[c].size() && st == JF_OK; ++q)
    st = joint(cp.blocks[q].first, cp.blocks[q].last, S.block_off[c][q], &cp.blocks[q]);
  return st;
}

// The streams of lanes 1 .. n - 1 and all lanes' events (made on first use, default priority).
jf_status lanes_of(jf_plan* p, int n, hipStream_t stream, hipStream_t* lane) {
  DevState& S = state_of(p);
  lane[0] = stream;
  for (int l = 0; n > 1 && l < n; ++l) {
    if (!S.ev_lane[l]) JF_HIP(hipEventCreateWithFlags(&S.ev_lane[l], hipEventDisableTiming));
    if (!l) continue;
    if (!S.lane_stream[l - 1]) JF_HIP(hipStreamCreateWithFlags(&S.lane_stream[l - 1], hipStreamNonBlocking));
    lane[l] = S.lane_stream[l - 1];
  }
  return JF_OK;
}

// Clear component c's output and walk its levels depth first: every prefix is computed once and
// kept in its level buffer while the Kraus operators of the next sliced site are iterated.
// lanes > 1: the variants of the first sliced level, with all below them, are dealt to that many
// lanes beside each other (a step of one of them is bound by its launch or by the 64 workgroups of
// its grid run), each with level buffers and barrier flags of its own; the launches go out to the
// lanes in turn.  A plan of 16 leaves of 2^16 elements takes 1265 us one leaf after another and 531 in
// four lanes; up to 720 with other plans' streams alive, where lanes can share a hardware queue.
jf_status enqueue_component(jf_plan* p, unsigned char* ws, unsigned char* bufs, hipStream_t stream, size_t c, Prof* prof,
                            Tune* tune, GridUse* gu, int lanes = 1) {
  const ComponentProgram& cp = p->prog.comps[c];
  DevState& S = state_of(p);
  const DevLayout& L = S.lay;
  // Every output entry is written by the final steps of the leaves, except where leaves add
  // partial traces into it (sliced wires) or a site's Kraus count is no power of two (padded
  // variants): only then is the output cleared first.
  bool clear = cp.accumulate;
  for (size_t site = 0; site < cp.out_bit.size() && site < p->prog.site_nk.size() && !clear; ++site) {
    const int nk = p->prog.site_nk[site];
    if (!cp.out_bit[site].empty() && (nk & (nk - 1))) clear = true;
  }
  if (clear) JF_HIP(launch_zero(ws + L.out_off + size_t(cp.out_off) * 16, cp.out_len, stream));
  struct Frame {
    int lv;
    int v, by;  // the variant and the distance to the lane's next one
    const void* parent;
    long long base;
  };
  const int split = first_sliced(cp);
  lanes = split < 0 || cp.accumulate ? 1 : std::min(lanes, cp.levels[split].nvar);
  hipStream_t lane[BATCH_LANES] = {stream};
  std::vector<int> vv[BATCH_LANES];  // the values of the levels on a lane's current path
  std::vector<Frame> stack[BATCH_LANES];
  if (lanes > 1) {
    const jf_status st = lanes_of(p, lanes, stream, lane);
    if (st != JF_OK) return st;
  }
  auto descend = [&](int l, int lv, const void* parent, long long base) -> jf_status {
    if (lv != split || lanes == 1) {
      stack[l].push_back({lv, 0, 1, parent, base});
      return JF_OK;
    }
    JF_HIP(hipEventRecord(S.ev_lane[0], stream));  // reached once: no level above it has variants
    for (int k = 0; k < lanes; ++k) {
      if (k) JF_HIP(hipStreamWaitEvent(lane[k], S.ev_lane[0], 0));
      stack[k].push_back({lv, k, lanes, parent, base});
    }
    return JF_OK;
  };
  for (auto& v : vv) v.assign(cp.levels.size(), 0);
  jf_status st = descend(0, 0, nullptr, 0);
  if (st != JF_OK) return st;
  for (bool more = true; more;) {
    more = false;
    for (int l = 0; l < lanes; ++l) {
      if (stack[l].empty()) continue;
      more = true;
      Frame f = stack[l].back();
      stack[l].pop_back();
      const Level& lev = cp.levels[f.lv];
      if (f.v + f.by < lev.nvar) stack[l].push_back({f.lv, f.v + f.by, f.by, f.parent, f.base});
      vv[l][f.lv] = f.v;
      const long long base = f.base + f.v * lev.out_stride;
      const void* cur = nullptr;
      if (gu) gu->lane = l;
      st = enqueue_level(p, ws, l ? ws + L.lane_off + size_t(l - 1) * L.lane_stride : bufs, lane[l], c, f.lv, vv[l],
                         f.parent, base, &cur, prof, tune, gu);
      if (st == JF_OK && f.lv + 1 < (int)cp.levels.size()) st = descend(l, f.lv + 1, cur, base);
      if (st != JF_OK) return st;
    }
  }
  for (int l = 1; l < lanes; ++l) {
    JF_HIP(hipEventRecord(S.ev_lane[l], lane[l]));
    JF_HIP(hipStreamWaitEvent(stream, S.ev_lane[l], 0));
  }
  return JF_OK;
}

// Enqueue the whole program (no synchronisation, no host copies): used eagerly and for capture.
// bufs: the level-buffer region (nullptr: the plan's own, at the end of its workspace).
// The plan's side stream and its fork / join events (created on first use, default priority).
jf_status side_of(jf_plan* p, hipStream_t* side) {
  DevState& S = state_of(p);
  // each object once (a failure part-way leaves the ones made for the next call to keep)
  if (!S.ev_fork) JF_HIP(hipEventCreateWithFlags(&S.ev_fork, hipEventDisableTiming));
  if (!S.ev_join) JF_HIP(hipEventCreateWithFlags(&S.ev_join, hipEventDisableTiming));
  if (!S.side_stream) JF_HIP(hipStreamCreateWithFlags(&S.side_stream, hipStreamNonBlocking));
  *side = S.side_stream;
  return JF_OK;
}

// Launch the persistent kernel over items on `side` (forked from and joined back to `stream` by
// fork / join; the caller waits on join) or, with no side stream, on `stream` itself.
jf_status launch_persistent_beside(const LdsItem* items, int n, const LdsStep* steps, hipStream_t stream,
                                   hipStream_t side, hipEvent_t fork, hipEvent_t join) {
  if (!side) {
    JF_HIP(launch_persistent(items, n, steps, stream));
    return JF_OK;
  }
  JF_HIP(hipEventRecord(fork, stream));
  JF_HIP(hipStreamWaitEvent(side, fork, 0));
  JF_HIP(launch_persistent(items, n, steps, side));
  JF_HIP(hipEventRecord(join, side));
  return JF_OK;
}

// Enqueue one whole pass of a plan.  side: a stream for the persistent launch of the small
// components, which then overlaps the other components' steps (one workgroup per component, so
// it leaves the rest of the device to them); null runs everything on `stream` in order.
// Arguments of the assembly of a plan's F_J from its component sums (device addresses in ws).
AssembleArgs assemble_args(jf_plan* p, unsigned char* ws, double* host) {
  const Program& P = p->prog;
  const DevState& S = state_of(p);
  const double s = std::exp2(P.log2_scale);  // exact: an integer power of two
  const cd v0 = s * P.scalar;
  AssembleArgs a;
  a.sums = reinterpret_cast<const double*>(ws + S.lay.sums_off);
  a.ncomp = int(P.comps.size());
  a.alg = P.opt.alg;
  a.a = s * s * std::norm(P.scalar);
  a.v0re = v0.real();
  a.v0im = v0.imag();
  a.res = reinterpret_cast<double*>(ws + S.lay.res_off);
  a.host = host;
  a.fail = reinterpret_cast<const unsigned*>(ws + S.lay.fail_off);
  a.counter = reinterpret_cast<unsigned*>(ws + S.lay.ctr_off);
  return a;
}

// The product over components and 1 - F_J of a plan, on the device (after all its components).
jf_status enqueue_assemble(jf_plan* p, unsigned char* ws, hipStream_t stream, double* host) {
  JF_HIP(launch_assemble(assemble_args(p, ws, host), stream));
  return JF_OK;
}

jf_status enqueue_program(jf_plan* p, unsigned char* ws, hipStream_t stream, double* host, Prof* prof = nullptr,
                          bool skip_lds = false, Tune* tune = nullptr, unsigned char* bufs = nullptr,
                          hipStream_t side = nullptr, bool assemble = true, bool grid = true, int lanes = 1) {
  const Program& P = p->prog;
  DevState& S = state_of(p);
  const DevLayout& L = S.lay;
  if (!bufs) bufs = ws + L.buf_off;
  S.grid_launches = S.grid_steps = 0;
  S.lanes = lanes;
  const bool lds = !skip_lds && !L.lds_comps.empty();
  if (lds && assemble && L.lds_comps.size() == P.comps.size()) {
    // every component in the persistent launch, which also assembles: one launch per run
    JF_HIP(launch_persistent_assemble(reinterpret_cast<const LdsItem*>(ws + L.lds_items_off),
                                      int(L.lds_comps.size()),
                                      reinterpret_cast<const LdsStep*>(ws + L.lds_steps_off),
                                      assemble_args(p, ws, host), stream));
    return JF_OK;
  }
  if (!lds) side = nullptr;
  if (lds) {
    const jf_status st = launch_persistent_beside(reinterpret_cast<const LdsItem*>(ws + L.lds_items_off),
                                                  int(L.lds_comps.size()),
                                                  reinterpret_cast<const LdsStep*>(ws + L.lds_steps_off), stream,
                                                  side, S.ev_fork, S.ev_join);
    if (st != JF_OK) return st;
  }
  grid = grid && L.grid && !S.grid_gave_up && grid_fits_device();
  size_t last = 0;  // the last component on this stream
  for (size_t c = 0; c < P.comps.size(); ++c)
    if (!P.comps[c].lds_resident) last = c;
  bool assembled = false;
  for (size_t c = 0; c < P.comps.size(); ++c) {
    const ComponentProgram& cp = P.comps[c];
    if (cp.lds_resident) continue;
    GridUse gu;
    gu.assemble = assemble && !side && c == last;
    gu.host = host;
    jf_status st = enqueue_component(p, ws, bufs, stream, c, prof, tune, grid ? &gu : nullptr, lanes);
    if (st != JF_OK) return st;
    if (!gu.summed)
      JF_HIP(launch_sumsq(ws + L.out_off + size_t(cp.out_off) * 16, cp.out_len,
                          reinterpret_cast<double*>(ws + L.sums_off) + 4 * c,
                          reinterpret_cast<double*>(ws + L.sumsq_off), stream));
    assembled = gu.assembled;
  }
  if (side) JF_HIP(hipStreamWaitEvent(stream, S.ev_join, 0));
  return assemble && !assembled ? enqueue_assemble(p, ws, stream, host) : JF_OK;
}

// Copy the plan's tables into ws (unless they are there already).  region: the bytes from ws on
// that the plan's runs write (0: its whole workspace); every other upload in it is forgotten.
jf_status upload(jf_plan* p, void* ws, hipStream_t stream, size_t region = 0) {
  DevState& S = state_of(p);
  if (!region) region = S.lay.total;
  std::lock_guard<std::mutex> g(g_upload_mu);
  if (S.uploaded_to == ws) {
    auto it = g_last_upload.find(ws);
    if (it != g_last_upload.end() && it->second.plan == p && it->second.bytes >= region) return JF_OK;
  }
  fill_lds_tables(p->prog, S.lay, static_cast<unsigned char*>(ws),
                  reinterpret_cast<LdsItem*>(&S.host_image[S.lay.lds_items_off]),
                  reinterpret_cast<LdsStep*>(&S.host_image[S.lay.lds_steps_off]), 0);
  JF_HIP(hipMemcpyAsync(ws, S.host_image.data(), S.host_image.size(), hipMemcpyHostToDevice, stream));
  JF_HIP(hipStreamSynchronize(stream));
  S.uploaded_to = ws;
  const auto a = reinterpret_cast<uintptr_t>(ws);
  forget_uploads(a, a + region);
  g_last_upload[ws] = Upload{p, region};
  return JF_OK;
}

jf_status check_ws(jf_plan* p, void* ws, size_t ws_bytes) {
  DevState& S = state_of(p);
  if (!S.validated) {
    std::string why;
    if (!validate_program(p->prog, why)) {
      set_error("plan failed validation: " + why);
      return JF_E_ARG;
    }
    S.validated = true;
  }
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255)) {
    set_error("workspace must be a 256-byte aligned device pointer");
    return JF_E_ARG;
  }
  if (ws_bytes < S.lay.total) {
    set_error("workspace of " + std::to_string(ws_bytes) + " bytes, plan needs " + std::to_string(S.lay.total));
    return JF_E_OOM;
  }
  return JF_OK;
}

// The plan's pinned landing area: 4 doubles per component (every read-back of sums fits in it).
jf_status pinned_sums(jf_plan* p, double** out) {
  DevState& S = state_of(p);
  if (!S.pinned_sums)
    JF_HIP(hipHostMalloc(reinterpret_cast<void**>(&S.pinned_sums),
                         std::max<size_t>(p->prog.comps.size(), 1) * 4 * sizeof(double), hipHostMallocDefault));
  *out = S.pinned_sums;
  return JF_OK;
}

// Coherent (fine-grained) pinned memory and its device address: kernels' stores reach the host
// without any cache flush, and the host reads them after a synchronisation.
jf_status pinned_coherent(size_t bytes, void** host, void** dev) {
  void *h = nullptr, *d = nullptr;
  JF_HIP(hipHostMalloc(&h, bytes, hipHostMallocCoherent));
  const hipError_t e = hipHostGetDevicePointer(&d, h, 0);
  if (e != hipSuccess || !d) {
    (void)hipHostFree(h);
    set_error(std::string("hipHostGetDevicePointer: ") + hipGetErrorString(e));
    return JF_E_HIP;
  }
  *host = h;
  *dev = d;
  return JF_OK;
}

constexpr long long kTermsWithRes = 254;   // traces that share the result's page
constexpr long long kTermChunk = 1 << 15;  // traces per half of the landing area (512 KB)

// The landing area of the result (and of few traces).
jf_status pinned_res_of(jf_plan* p) {
  DevState& S = state_of(p);
  if (S.res.host) return JF_OK;
  void *h = nullptr, *d = nullptr;
  const jf_status st = pinned_coherent(4 * sizeof(double) + kTermsWithRes * sizeof(double2), &h, &d);
  S.res = {static_cast<double*>(h), static_cast<double*>(d)};
  return st;
}

// The landing areas of a batch of n entries, kept by its first plan; growing them voids its captured
// lanes, which write the old ones.
jf_status batch_res_of(DevState& S, int n) {
  if (n <= S.batch_entries) return JF_OK;
  void *h = nullptr, *d = nullptr;
  const jf_status st = pinned_coherent(size_t(n) * 4 * sizeof(double), &h, &d);
  if (st != JF_OK) return st;
  if (S.batch_res.host) (void)hipHostFree(S.batch_res.host);
  S.batch_res = {static_cast<double*>(h), static_cast<double*>(d)};
  S.batch_entries = n;
  S.graph_lanes = 0;
  return JF_OK;
}

// Arguments of the traces' kernel; false where the plan does not fit them (the host gathers then).
bool term_args(jf_plan* p, unsigned char* ws, TermArgs& a) {
  const Program& P = p->prog;
  if (P.site_nk.size() > size_t(TERM_SITES) || P.comps.size() > size_t(TERM_COMPS)) return false;
  std::memset(&a, 0, sizeof(a));
  a.out = reinterpret_cast<const double2*>(ws + state_of(p).lay.out_off);
  a.sites = int(P.site_nk.size());
  a.comps = int(P.comps.size());
  const cd s = std::exp2(P.log2_scale) * P.scalar;
  a.re = s.real();
  a.im = s.imag();
  for (size_t c = 0; c < P.comps.size(); ++c) a.comp_off[c] = P.comps[c].out_off;
  for (size_t i = 0; i < P.site_nk.size(); ++i) {
    if (P.site_nk[i] < 1 || P.site_nk[i] > 16) return false;
    a.nk[i] = (unsigned char)P.site_nk[i];
    a.comp[i] = (unsigned char)(P.site_comp[i] < 0 ? 255 : P.site_comp[i]);
    if (P.site_comp[i] < 0) continue;
    const std::vector<int>& ob = P.comps[P.site_comp[i]].out_bit[i];
    if (ob.size() > 4) return false;
    for (size_t b = 0; b < 4; ++b) a.bit[i][b] = (unsigned char)(b < ob.size() ? ob[b] : 0);
  }
  return true;
}

// The landing area of the traces and its events (made on first use).
jf_status pinned_terms_of(jf_plan* p) {
  DevState& S = state_of(p);
  const long long n = std::min(p->prog.kraus_terms, 2 * kTermChunk);
  if (n > kTermChunk)
    for (hipEvent_t& e : S.ev_terms)
      if (!e) JF_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  if (S.pinned_terms || n <= kTermsWithRes) return JF_OK;
  void *h = nullptr, *d = nullptr;
  const jf_status st = pinned_coherent(size_t(n) * sizeof(double2), &h, &d);
  S.pinned_terms = static_cast<double2*>(h);
  S.pinned_terms_dev = static_cast<double2*>(d);
  return st;
}

// Wait for the run and read F_J back (with terms, also the per-tuple outputs).  With a landing
// area the assembly kernel has written the result there, so only the terms need a copy; without (the
// no-allocation entry point: no host allocation by the library), the result is copied into pageable
// host memory.
jf_status read_results(jf_plan* p, unsigned char* ws, hipStream_t stream, jf_result* out, double* terms,
                       const Landing& res_at, bool* gave_up) {
  const Program& P = p->prog;
  DevState& S = state_of(p);
  double res[4];
  const bool on_host = res_at.host != nullptr;
  unsigned char copied[kResBehindFail + sizeof(res)];  // the failure word and the result
  if (!on_host) JF_HIP(hipMemcpyAsync(copied, ws + S.lay.fail_off, sizeof(copied), hipMemcpyDeviceToHost, stream));
  // the traces: put in order on the device, chunk by chunk through a pinned landing area (half of it
  // fills while the other is copied out); without host allocations, gathered on the host
  TermArgs ta;
  const long long total = terms ? P.kraus_terms : 0;
  const bool on_device = terms && on_host && term_args(p, ws, ta);
  double2 *land = nullptr, *land_dev = nullptr;
  if (on_device) {
    const jf_status st = pinned_terms_of(p);
    if (st != JF_OK) return st;
    const bool with_res = total <= kTermsWithRes;
    land = with_res ? reinterpret_cast<double2*>(S.res.host + 4) : S.pinned_terms;
    land_dev = with_res ? reinterpret_cast<double2*>(S.res.dev + 4) : S.pinned_terms_dev;
    JF_HIP(launch_terms(ta, 0, std::min(total, kTermChunk), land_dev, stream));
    if (total > kTermChunk) JF_HIP(hipEventRecord(S.ev_terms[0], stream));
  }
  std::vector<std::vector<cd>> co;
  if (terms && !on_device) {
    for (auto& cp : P.comps) {
      std::vector<cd> v(size_t(cp.out_len));
      JF_HIP(hipMemcpyAsync(v.data(), ws + S.lay.out_off + size_t(cp.out_off) * 16, size_t(cp.out_len) * 16,
                            hipMemcpyDeviceToHost, stream));
      co.push_back(std::move(v));
    }
  }
  if (total > kTermChunk && on_device) JF_HIP(hipEventSynchronize(S.ev_terms[0]));
  else JF_HIP(hipStreamSynchronize(stream));
  unsigned failed = 0;
  if (!on_host) std::memcpy(&failed, copied, sizeof(failed));
  std::memcpy(res, on_host ? reinterpret_cast<unsigned char*>(res_at.host) : copied + kResBehindFail, sizeof(res));
  *gave_up = failed != 0 || res[3] != 0.0;
  if (*gave_up) return JF_OK;
  jf_result r;
  static_result(P, &r);
  r.fj = res[0];
  r.one_minus_fj = res[1];
  r.imag_residual = res[2];
  *out = r;
  if (terms && !on_device) gather_terms(P, co, terms);
  for (long long at = 0, half = 0; on_device && at < total; at += kTermChunk, half ^= 1) {
    const long long next = at + kTermChunk;
    if (next < total) {
      JF_HIP(launch_terms(ta, next, std::min(total - next, kTermChunk), land_dev + (half ^ 1) * kTermChunk, stream));
      JF_HIP(hipEventRecord(S.ev_terms[half ^ 1], stream));
    }
    if (at) JF_HIP(hipEventSynchronize(S.ev_terms[half]));
    std::memcpy(terms + 2 * at, land + half * kTermChunk, size_t(std::min(total - at, kTermChunk)) * sizeof(double2));
  }
  return JF_OK;
}

// Before a pass: its result is not there until its assembly has written it, and a pass that ends
// without one reads as void.
void await_result(const Landing& at) {
  if (at.host) static_cast<volatile double*>(at.host)[3] = 1.0;
}

// Wait for a pass and read it back; a pass whose grid runs gave up waiting (their workgroups were not
// resident together: the device was held by others) is run again with a launch per step, and so are
// the plan's later ones.  bufs and
// skip_lds as in enqueue_program (a batch member).
jf_status finish_pass(jf_plan* p, unsigned char* ws, hipStream_t stream, jf_result* out, double* terms,
                      const Landing& at, unsigned char* bufs = nullptr, bool skip_lds = false) {
  bool gave_up = false;
  jf_status st = read_results(p, ws, stream, out, terms, at, &gave_up);
  if (st != JF_OK || !gave_up) return st;
  st = leave_grid(p, ws, stream);
  if (st != JF_OK) return st;
  await_result(at);
  ++state_of(p).reruns;
  st = enqueue_program(p, ws, stream, at.dev, nullptr, skip_lds, nullptr, bufs, nullptr, true, false);
  if (st != JF_OK) return st;
  st = read_results(p, ws, stream, out, terms, at, &gave_up);
  if (st == JF_OK && gave_up) {
    set_error("the pass ended without a result");
    return JF_E_HIP;
  }
  return st;
}

// One run of a plan.  With JF_FLAG_GRAPH the step program is captured into a hipGraph on the first
// run for a (workspace, stream, kernel choice) and replayed after that (the per-step cost here is
// on the GPU side, so replay saves little; see the flag).  The null stream cannot be captured: then
// the plan's own stream runs the graph, ordered after the work already on the null stream.
jf_status run_one(jf_plan* p, void* ws, size_t ws_bytes, hipStream_t stream, jf_result* out, double* terms) {
  jf_status st = check_ws(p, ws, ws_bytes);
  if (st != JF_OK) return st;
  DevState& S = state_of(p);
  const bool graph = (p->prog.opt.flags & JF_FLAG_GRAPH) != 0;
  const int lanes = ws_bytes >= S.lay.lanes_total ? S.lay.slice_lanes : 1;
  st = upload(p, ws, stream, lanes > 1 ? S.lay.lanes_total : 0);
  if (st != JF_OK) return st;
  st = pinned_res_of(p);  // before any enqueue or capture: the assembly writes the result there
  if (st != JF_OK) return st;
  if (!S.ev0) {
    JF_HIP(hipEventCreate(&S.ev0));
    JF_HIP(hipEventCreate(&S.ev1));
    JF_HIP(hipEventCreateWithFlags(&S.ev_order, hipEventDisableTiming));
  }
  unsigned char* w = static_cast<unsigned char*>(ws);
  hipStream_t s = stream;
  if (graph && stream == nullptr) {
    if (!S.own_stream) JF_HIP(hipStreamCreateWithFlags(&S.own_stream, hipStreamNonBlocking));
    JF_HIP(hipEventRecord(S.ev_order, nullptr));
    JF_HIP(hipStreamWaitEvent(S.own_stream, S.ev_order, 0));
    s = S.own_stream;
  }
  hipStream_t side = nullptr;
  if (!S.lay.lds_comps.empty() && S.lay.lds_comps.size() < p->prog.comps.size()) {
    st = side_of(p, &side);
    if (st != JF_OK) return st;
  }
  if (graph && (!S.run_graph || S.run_graph_ws != ws || S.run_graph_stream != s || S.run_graph_gen != S.variant_gen)) {
    if (S.run_graph) {
      hipGraphExecDestroy(S.run_graph);
      S.run_graph = nullptr;
    }
    hipGraph_t g = nullptr;
    JF_HIP(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    st = enqueue_program(p, w, s, S.res.dev, nullptr, false, nullptr, nullptr, side);
    const hipError_t ce = hipStreamEndCapture(s, &g);
    if (st != JF_OK) {
      if (ce == hipSuccess && g) hipGraphDestroy(g);
      return st;
    }
    if (ce != hipSuccess) {
      set_error(std::string("hipStreamEndCapture: ") + hipGetErrorString(ce));
      return JF_E_HIP;
    }
    const hipError_t ie = hipGraphInstantiate(&S.run_graph, g, nullptr, nullptr, 0);
    hipGraphDestroy(g);
    if (ie != hipSuccess) {
      S.run_graph = nullptr;
      set_error(std::string("hipGraphInstantiate: ") + hipGetErrorString(ie));
      return JF_E_HIP;
    }
    S.run_graph_ws = ws;
    S.run_graph_stream = s;
    S.run_graph_gen = S.variant_gen;
  }
  JF_HIP(hipEventRecord(S.ev0, s));
  await_result(S.res);
  S.reruns = 0;
  if (graph) {
    JF_HIP(hipGraphLaunch(S.run_graph, s));
  } else {
    st = enqueue_program(p, w, s, S.res.dev, nullptr, false, nullptr, nullptr, side, true, true, lanes);
    if (st != JF_OK) {  // nothing still runs in a lane when the caller gets its workspace back
      for (int l = 1; l < lanes; ++l)
        if (S.lane_stream[l - 1]) (void)hipStreamSynchronize(S.lane_stream[l - 1]);
      return st;
    }
  }
  JF_HIP(hipEventRecord(S.ev1, s));
  jf_result r;
  st = finish_pass(p, w, s, &r, terms, S.res);
  if (st != JF_OK) return st;
  float ms = 0;
  JF_HIP(hipEventElapsedTime(&ms, S.ev0, S.ev1));
  r.seconds = ms * 1e-3;
  *out = r;
  return JF_OK;
}

}  // namespace

size_t plan_workspace_bytes(jf_plan* p) { return state_of(p).lay.lanes_total; }

}  // namespace jf

using namespace jf;

extern "C" jf_status jf_fidelity_alg1(jf_plan* p, void* ws, size_t ws_bytes, void* stream, jf_result* out,
                                      double* terms) {
  if (!p || !out || p->prog.opt.alg != 1) {
    set_error("jf_fidelity_alg1: NULL argument or not an Algorithm I plan");
    return JF_E_ARG;
  }
  return run_one(p, ws, ws_bytes, static_cast<hipStream_t>(stream), out, terms);
}

// ------------------------------------------------------------- no-allocation entry point ---
// Device scratch of jf_fidelity_noalloc: one copy per GPU, held until the process ends.  In host
// code the name `scratch` is a host-side stand-in, never a device address: the device address
// comes from hipGetSymbolAddress, taken once per device with that device current.
static __device__ __align__(256) unsigned char scratch[JF_NOALLOC_BYTES + kGridTableBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch (looked up on its first use on that device).
jf_status scratch_of_current_device(void** out) {
  int dev = 0;
  JF_HIP(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) {
    set_error("jf_fidelity_noalloc: device index " + std::to_string(dev) + " beyond the supported " +
              std::to_string(kMaxDevices));
    return JF_E_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> g(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    JF_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) {
      set_error("jf_fidelity_noalloc: hipGetSymbolAddress returned no address for the scratch");
      return JF_E_HIP;
    }
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return JF_OK;
}
}  // namespace

extern "C" jf_status jf_fidelity_noalloc(jf_plan* p, void* stream_v, jf_result* out, double* terms) {
  if (!p || !out || (p->prog.opt.alg != 1 && p->prog.opt.alg != 2)) {
    set_error("jf_fidelity_noalloc: NULL argument or no algorithm in the plan");
    return JF_E_ARG;
  }
  if (terms && p->prog.opt.alg != 1) {
    set_error("jf_fidelity_noalloc: per-term traces exist for Algorithm I plans only");
    return JF_E_ARG;
  }
  const size_t need = state_of(p).lay.total - state_of(p).lay.grid_bytes;  // the grid runs' tables have room beside
  if (need > JF_NOALLOC_BYTES) {
    set_error("jf_fidelity_noalloc: the plan needs a workspace of " + std::to_string(need) +
              " bytes; the no-allocation scratch holds " + std::to_string((size_t)JF_NOALLOC_BYTES));
    return JF_E_OOM;
  }
  void* ws = nullptr;
  jf_status st = scratch_of_current_device(&ws);
  if (st != JF_OK) return st;
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  st = check_ws(p, ws, JF_NOALLOC_BYTES + kGridTableBytes);
  if (st != JF_OK) return st;
  const auto t0 = std::chrono::steady_clock::now();
  st = upload(p, ws, stream);  // a copy of the plan's tables (every plan shares the scratch)
  if (st != JF_OK) return st;
  state_of(p).reruns = 0;
  st = enqueue_program(p, static_cast<unsigned char*>(ws), stream, nullptr);  // eager: no graph, no events
  if (st != JF_OK) return st;
  jf_result r;
  st = finish_pass(p, static_cast<unsigned char*>(ws), stream, &r, terms, Landing());
  if (st != JF_OK) return st;
  r.seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
  *out = r;
  return JF_OK;
}

extern "C" jf_status jf_stream_copy(const void* src, void* dst, size_t bytes, int bytes_per_lane, void* stream_v,
                                    double* ms) {
  if (ms && bytes == 0 && (bytes_per_lane == 8 || bytes_per_lane == 16)) {  // nothing to copy, no launch
    *ms = 0.0;
    return JF_OK;
  }
  if (!src || !dst || !ms || (bytes_per_lane != 8 && bytes_per_lane != 16) || bytes % size_t(bytes_per_lane) ||
      (reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst)) % 16) {
    set_error("jf_stream_copy: bad argument (16-byte aligned buffers, bytes a multiple of 8 or 16 bytes per lane)");
    return JF_E_ARG;
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  EventPair ev;
  JF_HIP(hipEventCreate(&ev.a));
  JF_HIP(hipEventCreate(&ev.b));
  JF_HIP(launch_stream_copy(src, dst, bytes, bytes_per_lane, stream, ev.a, ev.b));
  JF_HIP(hipEventSynchronize(ev.b));
  float t = 0;
  JF_HIP(hipEventElapsedTime(&t, ev.a, ev.b));
  *ms = t;
  return JF_OK;
}

extern "C" jf_status jf_profile_run(jf_plan* p, void* ws, size_t ws_bytes, void* stream_v, jf_profile* out) {
  if (!p || !out) {
    set_error("jf_profile_run: bad argument");
    return JF_E_ARG;
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  jf_status st = check_ws(p, ws, ws_bytes);
  if (st != JF_OK) return st;
  st = upload(p, ws, stream);
  if (st != JF_OK) return st;
  Prof prof;
  EventPair ev;
  JF_HIP(hipEventCreate(&ev.a));
  JF_HIP(hipEventCreate(&ev.b));
  hipEvent_t e0 = ev.a, e1 = ev.b;
  JF_HIP(hipEventRecord(e0, stream));
  st = enqueue_program(p, static_cast<unsigned char*>(ws), stream, nullptr, &prof);
  if (st != JF_OK) return st;
  JF_HIP(hipEventRecord(e1, stream));
  JF_HIP(hipStreamSynchronize(stream));
  jf_profile r = {};
  r.launches = (long long)prof.ev.size() / 2;
  for (size_t i = 0; i + 1 < prof.ev.size(); i += 2) {
    float ms = 0;
    JF_HIP(hipEventElapsedTime(&ms, prof.ev[i], prof.ev[i + 1]));
    r.kernel_ms += ms;
    r.max_launch_ms = std::max(r.max_launch_ms, double(ms));
  }
  float tot = 0;
  JF_HIP(hipEventElapsedTime(&tot, e0, e1));
  r.total_ms = tot;
  r.bytes = prof.bytes;
  r.flops = prof.flops;
  *out = r;
  return JF_OK;
}

extern "C" jf_status jf_profile_steps(jf_plan* p, void* ws, size_t ws_bytes, void* stream_v, jf_step_profile* out,
                                      int cap, int* n_launches) {
  if (!p || !n_launches || cap < 0 || (cap > 0 && !out)) {
    set_error("jf_profile_steps: bad argument");
    return JF_E_ARG;
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  jf_status st = check_ws(p, ws, ws_bytes);
  if (st != JF_OK) return st;
  st = upload(p, ws, stream);
  if (st != JF_OK) return st;
  Prof prof;
  st = enqueue_program(p, static_cast<unsigned char*>(ws), stream, nullptr, &prof);
  if (st != JF_OK) return st;
  JF_HIP(hipStreamSynchronize(stream));
  const int n = int(prof.rec.size());
  for (int i = 0; i < n; ++i) {
    float ms = 0;
    JF_HIP(hipEventElapsedTime(&ms, prof.ev[2 * i], prof.ev[2 * i + 1]));
    prof.rec[i].ms = ms;
    if (i < cap) out[i] = prof.rec[i];
  }
  *n_launches = n;
  return JF_OK;
}

extern "C" jf_status jf_autotune(jf_plan* p, void* ws, size_t ws_bytes, void* stream_v, int reps) {
  if (!p) {
    set_error("jf_autotune: bad argument");
    return JF_E_ARG;
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  jf_status st = check_ws(p, ws, ws_bytes);
  if (st != JF_OK) return st;
  st = upload(p, ws, stream);
  if (st != JF_OK) return st;
  state_of(p).grid_gave_up = false;
  state_of(p).joint_timings = 0;
  Tune tune;
  tune.reps = reps > 0 ? reps : 3;
  tune.done.resize(p->prog.comps.size());
  for (size_t c = 0; c < p->prog.comps.size(); ++c) tune.done[c].assign(p->prog.comps[c].steps.size(), 0);
  st = enqueue_program(p, static_cast<unsigned char*>(ws), stream, nullptr, nullptr, false, &tune);
  if (st != JF_OK) return st;
  JF_HIP(hipStreamSynchronize(stream));
  state_of(p).variant_gen = g_variant_gen.fetch_add(1);
  return JF_OK;
}

extern "C" jf_status jf_last_pass(jf_plan* p, jf_pass* out) {
  if (!p || !out) {
    set_error("jf_last_pass: bad argument");
    return JF_E_ARG;
  }
  const DevState& S = state_of(p);
  out->grid_launches = S.grid_launches;
  out->grid_steps = S.grid_steps;
  out->lanes = S.lanes;
  out->reruns = S.reruns;
  out->joint_timings = S.joint_timings;
  return JF_OK;
}

extern "C" jf_status jf_set_grid_wait(jf_plan* p, long long ticks) {
  if (!p || ticks < 0) {
    set_error("jf_set_grid_wait: bad argument");
    return JF_E_ARG;
  }
  DevState& S = state_of(p);
  S.grid_wait = ticks;
  S.grid_gave_up = false;
  S.variant_gen = g_variant_gen.fetch_add(1);  // captured launches hold the old limit
  return JF_OK;
}

extern "C" jf_status jf_set_kernel_variant(jf_plan* p, int variant) {
  if (!p || variant < KV_AUTO || variant >= KV_COUNT) {
    set_error("jf_set_kernel_variant: bad argument");
    return JF_E_ARG;
  }
  DevState& S = state_of(p);
  for (size_t c = 0; c < p->prog.comps.size(); ++c)
    for (size_t s = 0; s < p->prog.comps[c].steps.size(); ++s) {
      StepDesc* hd = reinterpret_cast<StepDesc*>(&S.host_image[S.lay.step_desc[c][s]]);
      hd->variant = variant_applies(*hd, variant) ? variant : KV_AUTO;
    }
  // a forced kernel runs every step on its own, except the Gauss-form kernels, whose products the
  // chains repeat; AUTO brings the chains back
  if (variant == KV_AUTO) S.grid_gave_up = false;
  const bool keep = variant == KV_AUTO || variant == KV_GAUSS_256 || variant == KV_GAUSS_512;
  for (auto& v : S.chain_off) std::fill(v.begin(), v.end(), char(!keep));
  for (auto* off : {&S.run_off, &S.block_off})
    for (auto& v : *off) std::fill(v.begin(), v.end(), char(variant != KV_AUTO));
  S.variant_gen = g_variant_gen.fetch_add(1);
  return JF_OK;
}

// Definition 1 decided with early stopping (Algorithm I, Section IV-A: the terms are
// nonnegative, so a running sum above 1 - eps proves equivalence).  Every component but the one
// with the most depth-first leaves runs in full; that one runs leaf by leaf.  After each leaf:
//   lower = a * prod_{other c} S_c * S_last(partial)           (the terms done so far)
//   upper = lower + (mass of the leaves not run) * prod_{sites outside} sum_j ||K_j||^2
// because |t_k|^2 = |tr(U^dagger E_k)|^2 / d^2 <= prod_i ||K_{k_i}||^2 for every Kraus tuple.
extern "C" jf_status jf_decide_equivalence(jf_plan* p, double eps, void* ws, size_t ws_bytes, void* stream_v,
                                           jf_decision* out) {
  if (!p || !out || !(eps > 0.0) || !(eps <= 1.0)) {
    set_error("jf_decide_equivalence: NULL argument or eps outside (0, 1]");
    return JF_E_ARG;
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  jf_status st = check_ws(p, ws, ws_bytes);
  if (st != JF_OK) return st;
  st = upload(p, ws, stream);
  if (st != JF_OK) return st;
  const Program& P = p->prog;
  const DevLayout& L = state_of(p).lay;
  unsigned char* w = static_cast<unsigned char*>(ws);
  // arithmetic margin of the form (the parity bar of its results)
  const double margin = P.opt.dtype == JF_C128 ? 1e-12 : 1e-6;
  const double thr = 1.0 - eps;
  jf_decision d = {};
  d.margin = margin;
  d.leaves_total = P.work_items;
  EventPair ev;
  JF_HIP(hipEventCreate(&ev.a));
  JF_HIP(hipEventCreate(&ev.b));
  hipEvent_t e0 = ev.a, e1 = ev.b;
  JF_HIP(hipEventRecord(e0, stream));
  auto decide = [&](double lo, double hi) {
    if (lo - margin > thr) return 1;
    if (hi + margin <= thr) return 0;
    return -1;
  };
  int last = -1;
  long long most = 1;
  bool wires = false;  // a leaf of a component with sliced wires holds partial sums, not terms
  for (const ComponentProgram& cp : P.comps) wires = wires || cp.accumulate;
  if (P.opt.alg == 1 && !wires)
    for (size_t c = 0; c < P.comps.size(); ++c)
      if (!P.comps[c].lds_resident && P.comps[c].leaves > most) {
        most = P.comps[c].leaves;
        last = int(c);
      }
  if (last < 0) {  // one pass computes every term
    st = pinned_res_of(p);
    if (st != JF_OK) return st;
    const Landing& at = state_of(p).res;
    await_result(at);
    state_of(p).reruns = 0;
    st = enqueue_program(p, w, stream, at.dev);
    if (st != JF_OK) return st;
    jf_result r;
    st = finish_pass(p, w, stream, &r, nullptr, at);
    if (st != JF_OK) return st;
    d.fj_lower = d.fj_upper = r.fj;
    d.leaves_run = d.leaves_total;
    d.decision = decide(r.fj, r.fj);
  } else {
    // everything except the last component, in full
    if (!L.lds_comps.empty())
      JF_HIP(launch_persistent(reinterpret_cast<const LdsItem*>(w + L.lds_items_off), int(L.lds_comps.size()),
                               reinterpret_cast<const LdsStep*>(w + L.lds_steps_off), stream));
    for (size_t c = 0; c < P.comps.size(); ++c) {
      const ComponentProgram& cp = P.comps[c];
      if (cp.lds_resident || int(c) == last) continue;
      st = enqueue_component(p, w, w + L.buf_off, stream, c, nullptr, nullptr, nullptr);
      if (st != JF_OK) return st;
      JF_HIP(launch_sumsq(w + L.out_off + size_t(cp.out_off) * 16, cp.out_len,
                          reinterpret_cast<double*>(w + L.sums_off) + 4 * c,
                          reinterpret_cast<double*>(w + L.sumsq_off), stream));
    }
    double* pin = nullptr;
    st = pinned_sums(p, &pin);
    if (st != JF_OK) return st;
    std::vector<double> sums(4 * P.comps.size());
    JF_HIP(hipMemcpyAsync(pin, w + L.sums_off, sums.size() * sizeof(double), hipMemcpyDeviceToHost, stream));
    JF_HIP(hipStreamSynchronize(stream));
    std::memcpy(sums.data(), pin, sums.size() * sizeof(double));
    const double sc = std::exp2(P.log2_scale);
    double prod_other = sc * sc * std::norm(P.scalar);
    for (size_t c = 0; c < P.comps.size(); ++c)
      if (int(c) != last) prod_other *= sums[4 * c] + sums[4 * c + 1];
    // masses: sites of the last component, and the rest
    const ComponentProgram& cp = P.comps[last];
    double mass_outside = 1.0, mass_unsliced = 1.0;
    std::vector<char> sliced(P.site_norm2.size(), 0);
    for (const Level& lev : cp.levels)
      if (lev.site >= 0) sliced[lev.site] = 1;
    for (size_t i = 0; i < P.site_norm2.size(); ++i) {
      double t = 0;
      for (double x : P.site_norm2[i]) t += x;
      if (P.site_comp[i] != last) mass_outside *= t;
      else if (!sliced[i]) mass_unsliced *= t;
    }
    double mass_total = mass_unsliced;
    for (const Level& lev : cp.levels)
      if (lev.site >= 0) {
        double t = 0;
        for (double x : P.site_norm2[lev.site]) t += x;
        mass_total *= t;
      }
    // the last component, leaf by leaf (depth first, prefixes kept in the level buffers)
    unsigned char* out_last = w + L.out_off + size_t(cp.out_off) * 16;
    double* sums_last = reinterpret_cast<double*>(w + L.sums_off) + 4 * last;
    JF_HIP(launch_zero(out_last, cp.out_len, stream));
    const int nl = int(cp.levels.size());
    std::vector<int> v(nl, 0);
    std::vector<const void*> end(nl, nullptr);
    std::vector<long long> base(nl, 0);
    int from = 0;
    double mass_done = 0;
    d.decision = -1;
    while (true) {
      for (int lv = from; lv < nl; ++lv) {
        base[lv] = (lv ? base[lv - 1] : 0) + v[lv] * cp.levels[lv].out_stride;
        st = enqueue_level(p, w, w + L.buf_off, stream, size_t(last), lv, v, lv ? end[lv - 1] : nullptr, base[lv], &end[lv],
                           nullptr, nullptr, nullptr);
        if (st != JF_OK) return st;
      }
      JF_HIP(launch_sumsq(out_last, cp.out_len, sums_last, reinterpret_cast<double*>(w + L.sumsq_off), stream));
      double part[2];
      JF_HIP(hipMemcpyAsync(pin, sums_last, sizeof(part), hipMemcpyDeviceToHost, stream));
      JF_HIP(hipStreamSynchronize(stream));
      std::memcpy(part, pin, sizeof(part));
      double m = mass_unsliced;
      for (int lv = 0; lv < nl; ++lv)
        if (cp.levels[lv].site >= 0) {
          const auto& nrm = P.site_norm2[cp.levels[lv].site];
          m *= v[lv] < int(nrm.size()) ? nrm[v[lv]] : 0.0;  // padding variants are zero operators
        }
      mass_done += m;
      ++d.leaves_run;
      d.fj_lower = prod_other * (part[0] + part[1]);
      d.fj_upper = d.fj_lower + std::max(0.0, mass_total - mass_done) * mass_outside;
      d.decision = decide(d.fj_lower, d.fj_upper);
      if (d.decision >= 0) break;
      // next leaf in depth-first order
      int lv = nl - 1;
      while (lv >= 0 && v[lv] + 1 >= cp.levels[lv].nvar) --lv;
      if (lv < 0) break;
      ++v[lv];
      for (int k = lv + 1; k < nl; ++k) v[k] = 0;
      from = lv;
    }
    d.leaves_run += P.work_items - cp.leaves;  // the other components ran in full
    if (d.leaves_run == P.work_items) d.fj_upper = d.fj_lower;  // every term is in
  }
  JF_HIP(hipEventRecord(e1, stream));
  JF_HIP(hipEventSynchronize(e1));
  float ms = 0;
  JF_HIP(hipEventElapsedTime(&ms, e0, e1));
  d.seconds = ms * 1e-3;
  *out = d;
  return JF_OK;
}

extern "C" jf_status jf_fidelity_alg2(jf_plan* p, void* ws, size_t ws_bytes, void* stream, jf_result* out) {
  if (!p || !out || p->prog.opt.alg != 2) {
    set_error("jf_fidelity_alg2: NULL argument or not an Algorithm II plan");
    return JF_E_ARG;
  }
  return run_one(p, ws, ws_bytes, static_cast<hipStream_t>(stream), out, nullptr);
}

// A batch shares one workspace: each plan keeps its tables, outputs and sums in a region of its
// own.  The members run in lanes beside each other, one after another within a lane: the level
// buffers of a lane's members share one region sized for the largest; the persistent kernel's item
// and step tables follow.  Most steps of small and medium members are bound by launches and by the
// few workgroups they have, so lanes overlap; a member with buffers beyond kLaneBytes fills the
// device by itself, and all of those share the first lane, so that the workspace grows by at most
// BATCH_LANES - 1 times kLaneBytes.  Longest members first, each to the lane with the least work.
// 40 uneven circuits of up to 11 qubits take 2474 us in one lane and 1457 in four (1549 launched call by
// call); up to 1930 with other plans' streams alive, where lanes can share a hardware queue.  As
// branches of one graph (its nodes are submitted branch after branch) they took 1822 us where a graph per
// lane took 1490.  96 circuits of four qubits took 320 us with an assembly launch each and 135 with one
// for all.
namespace jf {
namespace {
bool has_steps(jf_plan* p) { return state_of(p).lay.lds_comps.size() < p->prog.comps.size(); }

struct BatchLayout {
  std::vector<size_t> base;  // each plan's region
  std::vector<int> lane;     // each plan's lane
  size_t lane_bufs[BATCH_LANES] = {};
  size_t bufs = 0, items = 0, steps = 0, assembles = 0, total = 0;
};
BatchLayout batch_layout(jf_plan* const* plans, int n, int lanes) {
  BatchLayout b;
  size_t off = 0, items = 0, steps = 0;
  std::vector<int> order(n);
  for (int i = 0; i < n; ++i) {
    const DevLayout& L = state_of(plans[i]).lay;
    b.base.push_back(off);
    off += align256(L.buf_off);
    items += L.lds_comps.size();
    steps += L.lds_steps;
    order[i] = i;
  }
  auto buf_bytes = [&](int i) { return state_of(plans[i]).lay.total - state_of(plans[i]).lay.buf_off; };
  auto cost = [&](int i) { return has_steps(plans[i]) ? plans[i]->prog.est_seconds : 0.0; };
  std::stable_sort(order.begin(), order.end(), [&](int x, int y) {
    const bool bx = buf_bytes(x) > kLaneBytes, by = buf_bytes(y) > kLaneBytes;
    return bx != by ? bx : cost(x) > cost(y);
  });
  b.lane.assign(n, 0);
  double load[BATCH_LANES] = {};
  if (items) load[lanes - 1] = 3e-5;  // the persistent launch (20 to 50 us) runs ahead in the last lane
  size_t most[BATCH_LANES] = {};
  for (int i : order) {
    const int l = buf_bytes(i) > kLaneBytes ? 0 : int(std::min_element(load, load + lanes) - load);
    b.lane[i] = l;
    load[l] += cost(i);
    most[l] = std::max(most[l], buf_bytes(i));
  }
  b.bufs = off;
  for (int l = 0; l < lanes; ++l) {
    b.lane_bufs[l] = off;
    off += align256(most[l]);
  }
  b.items = off;
  off += align256(items * sizeof(LdsItem));
  b.steps = off;
  off += align256(steps * sizeof(LdsStep));
  b.assembles = off;
  off += align256(size_t(n) * sizeof(AssembleArgs));
  b.total = off;
  return b;
}
}  // namespace
}  // namespace jf

extern "C" jf_status jf_batch_workspace(jf_plan* const* plans, int n, size_t* bytes) {
  if (!plans || n < 0 || !bytes) {
    set_error("jf_batch_workspace: bad argument");
    return JF_E_ARG;
  }
  for (int i = 0; i < n; ++i)
    if (!plans[i]) {
      set_error("jf_batch_workspace: NULL plan");
      return JF_E_ARG;
    }
  *bytes = batch_layout(plans, n, BATCH_LANES).total;
  return JF_OK;
}

extern "C" jf_status jf_workspace_release(const void* dev_ws, size_t ws_bytes) {
  if (!dev_ws) {
    set_error("jf_workspace_release: NULL workspace");
    return JF_E_ARG;
  }
  // forget every upload whose region meets [dev_ws, dev_ws + ws_bytes): the plans whose tables
  // were there upload them again on their next call (batch members sit at offsets inside the range)
  const auto lo = reinterpret_cast<uintptr_t>(dev_ws);
  const auto hi = lo + (ws_bytes ? ws_bytes : 1);
  std::lock_guard<std::mutex> g(g_upload_mu);
  forget_uploads(lo, hi);
  return JF_OK;
}

extern "C" jf_status jf_fidelity_batch(jf_plan* const* plans, int n, void* ws, size_t ws_bytes, void* stream_v,
                                       jf_result* out) {
  size_t need = 0;
  jf_status st = jf_batch_workspace(plans, n, &need);
  if (st != JF_OK) return st;
  if (n == 0) return JF_OK;
  if (!out || !ws || (reinterpret_cast<uintptr_t>(ws) & 255)) {
    set_error("jf_fidelity_batch: bad output or workspace");
    return JF_E_ARG;
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_v);
  const int lanes = ws_bytes >= need ? BATCH_LANES : 1;
  const BatchLayout bl = batch_layout(plans, n, lanes);
  if (ws_bytes < bl.total) {
    set_error("jf_fidelity_batch: workspace too small");
    return JF_E_OOM;
  }
  unsigned char* w = static_cast<unsigned char*>(ws);
  {
    // the shared buffers and the persistent tables are written by this call: no plan's tables
    // uploaded there before survive it
    std::lock_guard<std::mutex> g(g_upload_mu);
    const auto a = reinterpret_cast<uintptr_t>(w + bl.bufs);
    forget_uploads(a, a + (bl.total - bl.bufs));
  }
  std::vector<unsigned char*> base(n);
  for (int i = 0; i < n; ++i) {
    base[i] = w + bl.base[i];
    st = check_ws(plans[i], base[i], state_of(plans[i]).lay.total);
    if (st != JF_OK) return st;
    st = upload(plans[i], base[i], stream, state_of(plans[i]).lay.buf_off);
    if (st != JF_OK) return st;
  }
  DevState& S0 = state_of(plans[0]);
  st = batch_res_of(S0, n);  // before the capture: each entry's assembly writes its result there
  if (st != JF_OK) return st;
  // every small component of every plan in one persistent launch, and one launch for the assembly
  // of all plans that have some
  std::vector<unsigned char> tables(bl.total - bl.items);
  LdsItem* items = reinterpret_cast<LdsItem*>(tables.data());
  LdsStep* lsteps = reinterpret_cast<LdsStep*>(tables.data() + (bl.steps - bl.items));
  AssembleArgs* assembles = reinterpret_cast<AssembleArgs*>(tables.data() + (bl.assembles - bl.items));
  int n_items = 0, n_lsteps = 0, n_assembles = 0;
  for (int i = 0; i < n; ++i) {
    const DevLayout& L = state_of(plans[i]).lay;
    fill_lds_tables(plans[i]->prog, L, base[i], items + n_items, lsteps + n_lsteps, n_lsteps);
    n_items += int(L.lds_comps.size());
    n_lsteps += L.lds_steps;
    if (!has_steps(plans[i]) || !L.lds_comps.empty())
      assembles[n_assembles++] = assemble_args(plans[i], base[i], S0.batch_res.entry(i).dev);
  }
  if (n_assembles) {
    JF_HIP(hipMemcpyAsync(w + bl.items, tables.data(), tables.size(), hipMemcpyHostToDevice, stream));
    JF_HIP(hipStreamSynchronize(stream));
  }
  EventPair ev;
  JF_HIP(hipEventCreate(&ev.a));
  JF_HIP(hipEventCreate(&ev.b));
  hipEvent_t e0 = ev.a, e1 = ev.b;
  // a lane of its own for the persistent launch where the members have only one
  bool used[BATCH_LANES] = {};
  bool large = false;
  for (int i = 0; i < n; ++i)
    if (has_steps(plans[i])) used[bl.lane[i]] = large = true;
  const int small_lane = !n_items ? -1 : !large ? 0 : lanes > 1 ? lanes - 1 : 1;
  if (small_lane >= 0) used[small_lane] = true;
  hipStream_t lane[BATCH_LANES] = {};
  int top = 0;  // lanes up to the last used one: a batch of small circuits makes no streams
  for (int l = 0; l < BATCH_LANES; ++l)
    if (used[l]) top = l;
  st = lanes_of(plans[0], top + 1, stream, lane);
  if (st != JF_OK) return st;
  // the launches of one lane, or of all (which = -1)
  auto enqueue_lane = [&](int which) -> jf_status {
    if (small_lane >= 0 && (which < 0 || which == small_lane))
      JF_HIP(launch_persistent(reinterpret_cast<const LdsItem*>(w + bl.items), n_items,
                               reinterpret_cast<const LdsStep*>(w + bl.steps), lane[small_lane]));
    for (int i = 0; i < n; ++i) {
      const int l = bl.lane[i];
      if ((which >= 0 && which != l) || !has_steps(plans[i])) continue;
      const jf_status ms =
          enqueue_program(plans[i], base[i], lane[l], S0.batch_res.entry(i).dev, nullptr, true, nullptr,
                          w + bl.lane_bufs[l], nullptr, state_of(plans[i]).lay.lds_comps.empty());
      if (ms != JF_OK) return ms;
    }
    return JF_OK;
  };
  std::vector<unsigned long long> key(n);
  for (int i = 0; i < n; ++i) key[i] = plans[i]->uid;
  std::vector<unsigned> gens(n);
  for (int i = 0; i < n; ++i) gens[i] = state_of(plans[i]).variant_gen;
  const bool graphs = stream != nullptr && large;
  if (graphs && (!S0.graph_lanes || S0.graph_ws != ws || S0.graph_stream != stream || S0.graph_plans != key ||
                 S0.graph_gens != gens || S0.graph_lanes != lanes)) {
    S0.graph_lanes = 0;
    for (int l = 0; l < BATCH_LANES; ++l) {
      if (S0.graph[l]) hipGraphExecDestroy(S0.graph[l]);
      S0.graph[l] = nullptr;
      if (!used[l]) continue;
      hipGraph_t g = nullptr;
      JF_HIP(hipStreamBeginCapture(lane[l], hipStreamCaptureModeThreadLocal));
      st = enqueue_lane(l);
      const hipError_t ce = hipStreamEndCapture(lane[l], &g);
      if (st != JF_OK) {
        if (ce == hipSuccess && g) hipGraphDestroy(g);
        return st;
      }
      if (ce != hipSuccess) {
        set_error(std::string("hipStreamEndCapture: ") + hipGetErrorString(ce));
        return JF_E_HIP;
      }
      const hipError_t ie = hipGraphInstantiate(&S0.graph[l], g, nullptr, nullptr, 0);
      hipGraphDestroy(g);
      if (ie != hipSuccess) {
        S0.graph[l] = nullptr;
        set_error(std::string("hipGraphInstantiate: ") + hipGetErrorString(ie));
        return JF_E_HIP;
      }
    }
    S0.graph_ws = ws;
    S0.graph_stream = stream;
    S0.graph_plans = key;
    S0.graph_gens = gens;
    S0.graph_lanes = lanes;
  }
  auto run = [&]() -> jf_status {
    for (int i = 0; i < n; ++i) {
      await_result(S0.batch_res.entry(i));
      state_of(plans[i]).reruns = 0;
    }
    JF_HIP(hipEventRecord(e0, stream));
    bool beside = false;
    for (int l = 1; l < BATCH_LANES; ++l) beside = beside || used[l];
    if (beside) JF_HIP(hipEventRecord(S0.ev_lane[0], stream));
    for (int l = 1; l < BATCH_LANES; ++l)
      if (used[l]) JF_HIP(hipStreamWaitEvent(lane[l], S0.ev_lane[0], 0));
    if (graphs) {
      for (int l = 0; l < BATCH_LANES; ++l)
        if (used[l]) JF_HIP(hipGraphLaunch(S0.graph[l], lane[l]));
    } else {
      const jf_status ls = enqueue_lane(-1);
      if (ls != JF_OK) return ls;
    }
    for (int l = 1; l < BATCH_LANES; ++l) {
      if (!used[l]) continue;
      JF_HIP(hipEventRecord(S0.ev_lane[l], lane[l]));
      JF_HIP(hipStreamWaitEvent(stream, S0.ev_lane[l], 0));
    }
    if (n_assembles)
      JF_HIP(launch_assembles(reinterpret_cast<const AssembleArgs*>(w + bl.assembles), n_assembles, stream));
    JF_HIP(hipEventRecord(e1, stream));
    return JF_OK;
  };
  st = run();
  if (st != JF_OK) {  // nothing still runs in a lane when the caller gets its workspace back
    for (hipStream_t l : lane)
      if (l) (void)hipStreamSynchronize(l);
    return st;
  }
  for (int i = 0; i < n; ++i) {
    st = finish_pass(plans[i], base[i], stream, &out[i], nullptr, S0.batch_res.entry(i), w + bl.lane_bufs[bl.lane[i]],
                     true);
    if (st != JF_OK) return st;
  }
  const int lanes_used = int(std::count(used, used + BATCH_LANES, true));
  for (int i = 0; i < n; ++i) state_of(plans[i]).lanes = lanes_used;
  float ms = 0;
  JF_HIP(hipEventElapsedTime(&ms, e0, e1));
  for (int i = 0; i < n; ++i) out[i].seconds = ms * 1e-3;
  return JF_OK;
}

extern "C" void jf_free_plan(jf_plan* p) {
  if (!p) return;
  if (p->dev) {
    auto* s = static_cast<DevState*>(p->dev);
    for (hipGraphExec_t g : s->graph)
      if (g) hipGraphExecDestroy(g);
    if (s->run_graph) hipGraphExecDestroy(s->run_graph);
    if (s->own_stream) {
      hipStreamSynchronize(s->own_stream);
      hipStreamDestroy(s->own_stream);
    }
    if (s->side_stream) {
      hipStreamSynchronize(s->side_stream);
      hipStreamDestroy(s->side_stream);
    }
    for (hipStream_t l : s->lane_stream)
      if (l) {
        hipStreamSynchronize(l);
        hipStreamDestroy(l);
      }
    for (hipEvent_t e : s->ev_lane)
      if (e) hipEventDestroy(e);
    for (hipEvent_t e : {s->ev0, s->ev1, s->ev_order, s->ev_fork, s->ev_join, s->ev_terms[0], s->ev_terms[1]})
      if (e) hipEventDestroy(e);
    if (s->pinned_sums) hipHostFree(s->pinned_sums);
    if (s->res.host) hipHostFree(s->res.host);
    if (s->batch_res.host) hipHostFree(s->batch_res.host);
    if (s->pinned_terms) hipHostFree(s->pinned_terms);
    {
      std::lock_guard<std::mutex> g(g_upload_mu);
      for (auto it = g_last_upload.begin(); it != g_last_upload.end();)
        if (it->second.plan == p) it = g_last_upload.erase(it);
        else ++it;
    }
    delete s;
  }
  delete p;
}
