// Host side of the C ABI: argument validation, buffer planning and the launch sequences.
// No device code lives here.  Validation never touches the HIP runtime, so every argument error
// can be produced on a machine without a GPU.
#include "../../include/lstm_abi.h"
#include "common.h"
#include "gemm_skinny.h"

#include <string.h>
#include <stdlib.h>
#include <algorithm>
#include <vector>

namespace lstm {
namespace {

constexpr size_t kAlign = 256;
constexpr unsigned kSpinLimit = 1u << 20;   // polls before a single-launch kernel's wait gives up (about a second)
inline size_t up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

struct Plan {
  int T, B, n_in, n, D;
  bool bf16;
  size_t esz;
  int nkc_f, nkc_b, nrt, ntile_f, ntile_b;
  int nkc_ll_f, ntile16;                    // ring layout of the single-launch forward kernels
  // reserve: per direction [gates float T*B*4n][hprev storage T*B*ldh], ldh = n rounded up to rows of whole 16-byte chunks
  long ldh;
  size_t res_gates, res_hprev, res_dir_stride, reserve_bytes;
  // workspace
  size_t ws_Wf, ws_Wb, ws_rows, ws_hfrag0, ws_hfrag1, ws_dzfrag0, ws_dzfrag1, ws_dzwide, ws_hstate, ws_cstate, ws_Dh, ws_Dc, ws_DZ, ws_Zx,
      ws_colsum, ws_sync, sync_bytes, ws_xpad, ws_fidx, ws_count, ws_Wcat, ws_Acat, ws_parts, parts_bytes, workspace_bytes;
  bool single_step, step_fused, step_few; int Kc, ksplit;         // T == 1 inference in bfloat16: the step is one product over [x | h], K cut in ksplit ranges
  bool small;                               // narrow layer: loop_small.hip
  bool blocks;                              // wide bfloat16 layer: loop_block.hip, if the device holds it
  size_t ws_blocks, ws_h0, ws_h0rows;
  bool zx_tiny, dw_tiny;                    // its products by gemm_tiny.hip
  size_t ws_tiny_cnt, ws_tiny_parts;
  bool zx_nn;                               // Zx of few 256 x 256 tiles: in K ranges (gemm_tile.hip)
  int n_in8;                                // n_in up to whole 16-byte chunks: row length of the padded copy of x there and for dW_x
  bool fast_gemm; int n_in_pad; long TBp;   // bf16 products through the kernels that load straight into LDS
  size_t hfrag_bytes, dzfrag_bytes, DZ_dir_elems, Zx_dir_elems, Wf_bytes;
};

// The products of a narrow layer (gemm_tiny.hip); sizes come from the plan alone, pointers from the call.
TinyProduct tiny_zx(const Plan& p, const void* x, const void* W_x, const void* b, float* gates, long gates_stride) {
  TinyProduct t = {};
  const long n4 = 4L * p.n;
  t.A = x; t.B = W_x; t.C = gates; t.bias = (const float*)b;
  t.M = p.T * p.B; t.N = (int)n4; t.K = p.n_in; t.lda = p.n_in; t.ldb = n4; t.ldc = n4;
  t.sBz = p.n_in * n4; t.sCz = gates_stride; t.sbiasz = n4; t.nz = p.D; t.nseg = 1; t.a_kcontig = 1;
  return t;
}
TinyGroup tiny_bwd(const Plan& p, const void* x, const void* W_x, const void* hprev, const void* DZ, const int32_t* lens, void* dx, void* dW_x,
                   void* dW_h, int acc) {
  TinyGroup g = {};
  const long n4 = 4L * p.n, hp_stride = (long)(p.res_dir_stride / p.esz);
  auto wgrad = [&](const void* A, long lda, long sAz, int M, void* C, const int32_t* mask) {
    TinyProduct t = {};
    t.A = A; t.B = DZ; t.C = C; t.M = M; t.N = (int)n4; t.K = p.T * p.B; t.lda = lda; t.ldb = n4; t.ldc = n4;
    t.sAz = sAz; t.sBz = (long)p.DZ_dir_elems; t.sCz = M * n4; t.nz = p.D; t.nseg = 1; t.accumulate = acc;
    t.lens = mask; t.Bt = p.B; t.T = p.T;
    return t;
  };
  g.p[g.count++] = wgrad(x, p.n_in, 0, p.n_in, dW_x, lens);     // (x may hold anything at padded frames; hprev and DZ are numbers there, DZ zeros)
  g.p[g.count++] = wgrad(hprev, p.ldh, hp_stride, p.n, dW_h, nullptr);
  if (dx) {
    TinyProduct t = {};
    t.A = DZ; t.B = W_x; t.C = dx; t.M = p.T * p.B; t.N = p.n_in; t.K = (int)n4; t.lda = n4; t.ldb = n4; t.ldc = p.n_in;
    t.nz = 1; t.nseg = p.D; t.sAseg = (long)p.DZ_dir_elems; t.sBseg = p.n_in * n4; t.a_kcontig = t.b_kcontig = 1; t.out_bf16 = p.bf16;
    g.p[g.count++] = t;
  }
  return g;
}

int make_plan(const lstm_desc* d, int bidir, Plan* p, bool odd_fast = true) {
  if (!d) return LSTM_ERR_NULL;
  if (d->T < 0 || d->B < 0 || d->n_in < 1 || d->n < 1) return LSTM_ERR_DIM;
  const long TB = (long)d->T * d->B;
  if (TB >= (1L << 31) || (long)d->n * 4 >= (1L << 29) || d->n_in >= (1 << 29) || d->B >= (1 << 24)) return LSTM_ERR_DIM;
  if (d->dtype != LSTM_F32 && d->dtype != LSTM_BF16_F32STATE) return LSTM_ERR_UNSUPPORTED;
  if (d->flags & ~(LSTM_FLAG_ACCUMULATE | LSTM_FLAG_PER_STEP | LSTM_FLAG_INFERENCE | LSTM_FLAG_WEIGHTS_PACKED | LSTM_FLAG_PLAIN_LAUNCH)) return LSTM_ERR_UNSUPPORTED;
  if (d->reserved != 0) return LSTM_ERR_UNSUPPORTED;
  p->T = d->T; p->B = d->B; p->n_in = d->n_in; p->n = d->n; p->D = bidir ? 2 : 1;
  p->bf16 = d->dtype == LSTM_BF16_F32STATE;
  p->esz = p->bf16 ? 2 : 4;
  const int KC = p->bf16 ? 32 : 16;                 // k covered by one fragment chunk index
  p->nkc_f = cdiv(d->n, KC);
  p->nkc_b = cdiv(4L * d->n, KC);
  p->nrt = 2 * cdiv(d->B > 0 ? d->B : 1, 32);       // 16-row tiles, two per work-group row block
  p->ntile_f = cdiv(d->n, 8);
  p->ntile_b = cdiv(d->n, 16);
  p->ntile16 = cdiv(d->n, 16);
  p->nkc_ll_f = ll_nkc(d->n, kLLSlotsFwd);
  const size_t n = d->n, D = p->D, B = d->B;
  const bool infer = d->flags & LSTM_FLAG_INFERENCE;
  p->res_gates = 0;
  p->res_hprev = up(TB * 4 * n * 4);
  p->ldh = p->bf16 ? (d->n + 7) / 8 * 8 : (d->n + 3) / 4 * 4;
  p->res_dir_stride = p->res_hprev + up(TB * p->ldh * p->esz);
  p->reserve_bytes = D * p->res_dir_stride + kAlign;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += up(bytes); return at; };
  // error word, per-row-tile words, then one word per work-group of a single-launch kernel (its XCD)
  p->sync_bytes = up((64 + 2 * (size_t)p->nrt) * 4 + std::max(D * 2 * (size_t)p->nrt * cdiv(d->n, 32), (size_t)256) * 4);
  p->ws_sync = take(p->sync_bytes);              // first, so that lstm_sync_status() finds it without a plan
  p->Wf_bytes = D * std::max((size_t)p->ntile_f * 2 * p->nkc_f * 1024, ll_wf_bytes(d->n, p->nkc_ll_f));
  p->ws_Wf = take(p->Wf_bytes + 1024);            // packed W_h, then one chunk of zeros
  const bool part = p->bf16 && d->n <= 1024;          // the partial-sum backward kernel may be chosen
  // float storage: the single-launch backward kernel (batches of up to 256 rows: its rings grow with B n^2 / 16)
  const bool part32 = !p->bf16 && d->n <= 1024 && d->B <= 256;
  p->ws_Wb = take(infer ? 0 : D * std::max({(size_t)p->ntile_b * p->nkc_b * 1024, part ? bwdp_wh_bytes(d->n, bwdp_nct(d->n)) : (size_t)0,
                                            part32 ? bwd_f32_wh_bytes(d->n) : (size_t)0}));
  p->hfrag_bytes = D * p->nrt * (size_t)std::max(p->nkc_f, p->nkc_ll_f) * 1024;
  p->dzfrag_bytes = D * std::max({p->nrt * (size_t)p->nkc_b * 1024, part ? bwdp_ring_bytes(d->B, d->n) : (size_t)0,
                                  part32 ? bwd_f32_ring_bytes(d->B, d->n) : (size_t)0});
  p->ws_hfrag0 = take(p->hfrag_bytes);
  p->ws_hfrag1 = take(p->hfrag_bytes);
  p->ws_dzfrag0 = take(infer ? 0 : p->dzfrag_bytes);
  p->ws_dzfrag1 = take(infer ? 0 : p->dzfrag_bytes);
  p->ws_dzwide = take(!infer && part32 ? D * bwd_f32_ring_bytes(d->B, d->n) : 0);
  p->ws_hstate = take(D * B * n * 4);
  p->ws_cstate = take(D * B * n * 4);
  p->ws_Dh = take(infer ? 0 : D * B * n * 4);
  p->ws_Dc = take(infer ? 0 : D * B * n * 4);
  p->DZ_dir_elems = up(TB * 4 * n * p->esz) / p->esz;
  p->ws_DZ = take(infer ? 0 : D * p->DZ_dir_elems * p->esz);
  p->Zx_dir_elems = up(TB * 4 * n * 4) / 4;
  // T == 1 inference, bfloat16: few output tiles, so K is cut into ranges that separate work-groups multiply (each at
  // least four 64-wide stages); their partial products lie side by side and the cell kernel adds them
  const bool fast = p->bf16 && (odd_fast || d->n % 2 == 0);
  p->single_step = fast && infer && d->T == 1 && !(d->flags & LSTM_FLAG_PER_STEP);
  // k extent of the input projection: a multiple of 8 (16-byte rows), and for narrow inputs a multiple of 64 so that
  // the product runs through the kernel that loads straight into LDS (x is then copied into zero-padded rows)
  p->n_in_pad = d->n_in < 256 ? (d->n_in + 63) / 64 * 64 : (d->n_in + 7) / 8 * 8;
  // The step's product has few rows: a work-group of the skinny-row kernel walks the whole K and applies the cell in its
  // epilogue (B <= kSkinnyMaxRows); larger batches go through the throughput kernel, K cut into ranges whose partial
  // products lie side by side for the cell kernel to add.
  p->step_fused = p->single_step && d->B <= kSkinnyMaxRows;
  p->step_few = p->step_fused && few_cell_pays(d->B, d->n, p->D, (long)p->n_in_pad + d->n);
  {
    const long tiles = (long)cdiv(B > 0 ? B : 1, 256) * cdiv(4L * d->n, 256) * p->D;
    const long stages = cdiv((long)p->n_in_pad + d->n, 64);
    p->ksplit = p->step_fused ? 1 : (int)std::max(1L, std::min(std::min(256 / tiles, stages / 4), 8L));
    p->Kc = cdiv((long)p->n_in_pad + d->n, 64L * p->ksplit) * 64 * p->ksplit;
  }
  p->ws_Zx = take(infer && !p->step_fused ? D * p->Zx_dir_elems * 4 * (p->single_step ? p->ksplit : 1) : 0);
  p->ws_colsum = take(infer ? 0 : D * 64 * 4 * n * 4);
  // padded operand copies for the fast bf16 products
  p->fast_gemm = fast;
  p->TBp = (TB + 63) / 64 * 64;
  const bool fg = p->fast_gemm;
  p->n_in8 = p->bf16 ? (d->n_in + 7) / 8 * 8 : (d->n_in + 3) / 4 * 4;
  p->zx_nn = fg && gemm_tile_small(TB, 4L * d->n, p->D);
  p->ws_xpad = take(fg || !p->bf16 ? TB * std::max(fg && !p->zx_nn && p->n_in_pad != d->n_in ? p->n_in_pad : 0, p->n_in8 != d->n_in ? p->n_in8 : 0) * p->esz : 0);
  // frame map of the batch (which frames are real), used to leave padded frames out of the products
  const bool fm = fg || !p->bf16;             // (float storage: its product kernels take the same row maps)
  p->ws_fidx = take(fm ? (size_t)p->TBp * 4 : 0);
  p->ws_count = take(fm ? 256 : 0);
  p->ws_Wcat = take(p->single_step ? D * std::max((size_t)4 * n, wcell_rows(d->n)) * p->Kc * 2 : 0);
  p->ws_Acat = take(p->single_step ? D * std::max((size_t)B * p->Kc * 2, frag_bytes(d->B, p->Kc)) : 0);
  // products with few output tiles: K ranges, whose parts gemm_tile.hip and gemm_float.hip sum
  const auto tile_parts = [&](long M, long N, long K, int nz, int nseg, bool frames) {
    if (!p->bf16) return gemm_float_parts_bytes(M, N, K, nz, nseg, frames);
    return fg && gemm_tile_small(M, N, nz) ? gemm_tile_parts_bytes(M, N, K, nz, nseg) : (size_t)0;
  };
  size_t tp = TB > 0 && (p->zx_nn || !p->bf16) && !p->single_step ? tile_parts(TB, 4L * d->n, p->n_in8, p->D, 1, true) : 0;
  if (TB > 0) tp = std::max(tp, tile_parts(d->B, 4L * d->n, p->ldh, 1, 1, false));      // (h0 W_h)
  if (!infer && TB > 0)                   // (the backward products' are added together at the end)
    tp = std::max(tp, up(tile_parts(TB, d->n_in, 4L * d->n, 1, p->D, true)) + up(std::max(tile_parts(d->n_in, 4L * d->n, TB, p->D, 1, false), fg ? gemm_tn_parts_bytes(d->n_in, 4L * d->n, TB, p->D) : 0)) +
                          up(std::max(tile_parts(d->n, 4L * d->n, TB, p->D, 1, false), fg ? gemm_tn_parts_bytes(d->n, 4L * d->n, TB, p->D) : 0)));
  p->parts_bytes = tp;
  p->ws_parts = take(p->parts_bytes);
  p->blocks = p->bf16 && loop_block_width(d->n) && !(d->flags & LSTM_FLAG_PER_STEP) && d->T >= 2 && TB > 0;
  p->ws_blocks = take(p->blocks ? loop_block_wh_bytes(d->n) + std::max(loop_block_ring_bytes(d->n), loop_block_ring_bytes_bwd(d->n)) : 0);
  // tables of rows one behind the other (whatever the device's size makes of them)
  p->ws_rows = take(p->bf16 && d->n <= 1024 && d->B > 8 && d->B <= kPackMaxRows ? 2 * (TB + kPackMaxSlots * ((size_t)d->T + 1)) * 4 + kPackMaxSlots / 8 * 4 : 0);
  p->ws_h0 = take(D * B * p->ldh * p->esz);
  p->ws_h0rows = take(D * B * 4);
  // (one step runs as one step of LSTM_FLAG_PER_STEP does, bit for bit)
  p->small = loop_small_ok(d->n) && !(d->flags & LSTM_FLAG_PER_STEP) && d->T >= 2 && TB > 0;
  p->zx_tiny = p->small && tiny_macs(tiny_zx(*p, nullptr, nullptr, nullptr, nullptr, 0)) <= kTinyZxMacs;
  p->dw_tiny = false;
  p->ws_tiny_cnt = p->ws_tiny_parts = o;
  if (p->small && !infer) {
    char any;
    const TinyGroup g = tiny_bwd(*p, nullptr, nullptr, nullptr, nullptr, nullptr, &any, nullptr, nullptr, 0);
    long macs = 0;
    for (int i = 0; i < g.count; ++i) macs += tiny_macs(g.p[i]);
    p->dw_tiny = macs <= kTinyBwdMacs;
    if (p->dw_tiny) {
      p->ws_tiny_cnt = take((size_t)tiny_counters(g) * 4);
      p->ws_tiny_parts = take(tiny_parts_bytes(g));
    }
  }
  p->workspace_bytes = o + kAlign;
  return LSTM_OK;
}

// The plan of a call that brings its buffers.  Workspaces of odd widths were smaller while their products took the generic kernel: such a one still serves, that way.
int call_plan(const lstm_desc* d, int bidir, Plan* p) {
  const int rc = make_plan(d, bidir, p);
  return !rc && p->bf16 && p->n % 2 != 0 && d->workspace_bytes < p->workspace_bytes ? make_plan(d, bidir, p, false) : rc;
}

bool misaligned(const void* p) { return ((uintptr_t)p & 15u) != 0; }

// rows one behind the other: the tables' places in the workspace
PackRows pack_rows(const Plan& p, char* ws, const int* lens, bool backward, const lstm_desc* desc) {
  PackRows r = {};
  if (!p.bf16 || p.n % 2 != 0 || !lens || p.B <= 8 || p.T < 2 || (desc->flags & LSTM_FLAG_PER_STEP)) return r;
  r.slots = persist_pack_slots(p.T, p.B, p.n, p.D, backward);
  if (r.slots == 0) return r;
  r.lens = lens; r.T = p.T; r.B = p.B; r.tab_steps = pack_tab_steps(p.T, p.B, r.slots); r.max_steps = pack_max_steps(p.T, backward);
  r.up = (unsigned*)(ws + p.ws_rows);
  r.down = r.up + (size_t)r.slots * r.tab_steps;
  r.steps = (int*)(r.down + (size_t)r.slots * r.tab_steps);
  return r;
}

int check_device() {                 // is the current device one this library is built for?  (looked up once per device)
  static std::atomic<unsigned long long> known_good{0};
  const hipError_t e = once_per_device(known_good, [] {
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return hipErrorInvalidDevice;
    return strncmp(prop.gcnArchName, "gfx950", 6) == 0 ? hipSuccess : hipErrorInvalidDevice;
  });
  if (e != hipSuccess) { (void)hipGetLastError(); return LSTM_ERR_HIP; }
  return 0;
}

// ---- optional phase timing (hipEvents on the caller's stream) -----------------------------------
// A bracket's time belongs to one phase, or to several that share its launches, in proportion to `weight`.
struct PhaseShare { int phase; double weight; };
struct PhaseRec { PhaseShare share[4]; int count; long launches; hipEvent_t e0, e1; };
int g_profile = 0;              // 0 off, 1 recurrent loops and hoisted products, 2 every phase
std::vector<PhaseRec> g_recs;

struct Phase {
  int idx = -1;
  hipStream_t s;
  Phase(int phase, long launches, hipStream_t stream) : Phase(std::initializer_list<PhaseShare>{{phase, 1.0}}, launches, stream) {}
  Phase(std::initializer_list<PhaseShare> shares, long launches, hipStream_t stream) : s(stream) {
    if (!g_profile) return;
    PhaseRec r = {};
    // (an event between two kernels leaves the device idle for some microseconds: the short set-up phases are
    // bracketed only on request)
    bool wanted = g_profile >= 2;
    for (const PhaseShare& p : shares) {
      if (p.weight <= 0.0 || r.count == 4) continue;
      r.share[r.count++] = p;
      wanted |= p.phase != LSTM_PHASE_PREP && p.phase != LSTM_PHASE_DB;
    }
    if (!wanted || r.count == 0) return;
    r.launches = launches;
    if (hipEventCreate(&r.e0) != hipSuccess || hipEventCreate(&r.e1) != hipSuccess) { (void)hipGetLastError(); return; }
    (void)hipEventRecord(r.e0, s);
    g_recs.push_back(r);
    idx = (int)g_recs.size() - 1;
  }
  ~Phase() { if (idx >= 0) (void)hipEventRecord(g_recs[idx].e1, s); }
};

#define HIPCHK(expr) do { if ((expr) != hipSuccess) { (void)hipGetLastError(); return LSTM_ERR_HIP; } } while (0)

int run_fwd(const lstm_desc* desc, int bidir, const void* x, const void* W_x, const void* W_h, const void* b,
            const void* h0, const void* c0, const int32_t* seq_lens, void* y, void* c, void* hT, void* cT, void* reserve,
            void* workspace, void* stream) {
  Plan p;
  int rc = call_plan(desc, bidir, &p);
  if (rc) return rc;
  if (!bidir && desc->direction != 1 && desc->direction != -1) return LSTM_ERR_DIRECTION;
  const bool infer = desc->flags & LSTM_FLAG_INFERENCE;
  if (!x || !W_x || !W_h || !y || !workspace) return LSTM_ERR_NULL;
  if (!infer && (!reserve || !c)) return LSTM_ERR_NULL;
  const void* ptrs[] = {x, W_x, W_h, b, h0, c0, seq_lens, y, c, hT, cT, reserve, workspace};
  for (const void* q : ptrs) if (misaligned(q)) return LSTM_ERR_ALIGN;
  if (desc->workspace_bytes < p.workspace_bytes) return LSTM_ERR_SIZE;
  if (!infer && desc->reserve_bytes < p.reserve_bytes) return LSTM_ERR_SIZE;
  if (p.B == 0) return LSTM_OK;
  if ((rc = check_device())) return rc;

  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)(((uintptr_t)workspace + kAlign - 1) / kAlign * kAlign);
  char* rs = reserve ? (char*)(((uintptr_t)reserve + kAlign - 1) / kAlign * kAlign) : nullptr;
  const size_t n = p.n, B = p.B, D = p.D, T = p.T;
  float* hstate = (float*)(ws + p.ws_hstate);
  float* cstate = (float*)(ws + p.ws_cstate);
  const size_t state_bytes = D * B * n * 4;

  if (p.single_step) {
    // the stepped cell: z = [x | h] [W_x ; W_h] + b as one product over all rows, then the cell update
    const long Kc = p.Kc;
    char* Wcat = ws + p.ws_Wcat;
    char* Acat = ws + p.ws_Acat;
    unsigned* status = (unsigned*)(ws + p.ws_sync);
    float* z = (float*)(ws + p.ws_Zx);
    if (p.step_few) {                  // a handful of rows: operands in fragment order
      if (!(desc->flags & LSTM_FLAG_WEIGHTS_PACKED)) {
        Phase ph(LSTM_PHASE_PREP, 1, s);
        HIPCHK(launch_pack_cell_frag(W_x, W_h, Wcat, p.n_in, p.n_in_pad, p.n, p.n_in_pad + p.n, p.D, s));
      }
      Phase ph(LSTM_PHASE_LOOP_FWD, 2, s);
      HIPCHK(launch_few_cell(x, (const float*)h0, Acat, Wcat, (const float*)b, (const float*)c0, (float*)hT, (float*)cT, y, (long)(D * n), (float*)c,
                             seq_lens, status, p.B, p.n_in, p.n_in_pad, p.n, p.D, s));
      return LSTM_OK;
    }
    {
      Phase ph(LSTM_PHASE_PREP, 2, s);
      if (!(desc->flags & LSTM_FLAG_WEIGHTS_PACKED)) {
        if (p.step_fused) HIPCHK(launch_pack_wcell(W_x, W_h, Wcat, p.n_in, p.n_in_pad, p.n, p.Kc, p.D, s));
        else HIPCHK(launch_pack_wcat(W_x, W_h, Wcat, p.n_in, p.n_in_pad, p.n, p.Kc, p.D, s));
      }
      HIPCHK(launch_concat_xh(x, (const float*)h0, Acat, p.B, p.n_in, p.n_in_pad, p.n, p.Kc, p.D, s));
    }
    if (p.step_fused) {                // product, bias, cell update and outputs in one kernel
      Phase ph(LSTM_PHASE_LOOP_FWD, 1, s);
      HIPCHK(launch_step_cell(Acat, Wcat, (const float*)b, (const float*)h0, (const float*)c0, (float*)hT, (float*)cT, y, (long)(D * n),
                              (float*)c, seq_lens, status, p.B, p.n, p.Kc, p.D, s));
      return LSTM_OK;
    }
    // batch index of the product = K range: A and B advance by Kr columns, C by one partial result
    const long Kr = Kc / p.ksplit, part = (long)p.Zx_dir_elems;
    {
      Phase ph(LSTM_PHASE_GEMM_ZX, (long)D, s);
      for (size_t d = 0; d < D; ++d) {
        GemmArgs g = {};
        g.A = Acat + d * B * Kc * 2; g.B = Wcat + d * (4 * n) * Kc * 2; g.C = z + d * p.ksplit * part;
        g.M = p.B; g.N = 4 * p.n; g.K = (int)Kr; g.lda = Kc; g.ldb = Kc; g.ldc = 4 * n;
        g.sAz = Kr; g.sBz = Kr; g.sCz = part; g.nz = p.ksplit; g.nseg = 1;
        g.a_kcontig = true; g.b_kcontig = true; g.in_bf16 = true; g.out_bf16 = false;
        // (ranges planned for that kernel's tiles: the one for few tiles takes 82 instead of 73 us a step at 1500 rows, 131 instead of 119 at 3000)
        HIPCHK(gemm_nt_ok(g) ? launch_gemm_nt(g, s) : launch_gemm(g, s));
      }
    }
    {
      Phase ph(LSTM_PHASE_LOOP_FWD, 1, s);
      HIPCHK(launch_cell_step(z, part, p.ksplit, (const float*)b, (const float*)h0, (const float*)c0, (float*)hT, (float*)cT, y,
                              (long)(D * n), (float*)c, seq_lens, status, p.B, p.n, p.D, s));
    }
    return LSTM_OK;
  }
  // hoisted input projection for all frames and both directions: Zx = X W_x + b
  float* gates = infer ? (float*)(ws + p.ws_Zx) : (float*)(rs + p.res_gates);
  const long gates_stride = infer ? (long)p.Zx_dir_elems : (long)(p.res_dir_stride / 4);
  bool frames_mapped = false;            // the frame map was written by the set-up launch
  auto projection = [&]() {
    GemmArgs g = {};
    g.A = x; g.B = W_x; g.C = gates; g.bias = (const float*)b;
    g.M = (int)(T * B); g.N = 4 * p.n; g.K = p.n_in;
    g.lda = p.n_in; g.ldb = 4 * n; g.ldc = 4 * n;
    g.sAz = 0; g.sBz = (long)p.n_in * 4 * n; g.sCz = gates_stride; g.sbiasz = 4 * n; g.nz = p.D; g.frames = true;
    g.nseg = 1; g.a_kcontig = true; g.b_kcontig = false; g.in_bf16 = p.bf16; g.out_bf16 = false;
    return g;
  };
  bool projected = false;                // the set-up launch did it
  bool x_padded = false;                 // likewise
  const int ldx = !p.bf16 ? p.n_in8 : !p.fast_gemm ? p.n_in : p.zx_nn ? p.n_in8 : p.n_in_pad;      // (bfloat16: rows of x are not 16-byte aligned, or narrow: zero-padded copy)
  // float storage: the product over padded rows, if the float kernel takes it
  auto padded_float = [&](GemmArgs g) {
    g.A = ws + p.ws_xpad; g.K = p.n_in8; g.lda = p.n_in8; g.k_phys_rows = p.n_in;
    return g;
  };
  auto project = [&]() -> int {
    if (projected) return LSTM_OK;
    GemmArgs g = projection();
    {
      Phase ph(LSTM_PHASE_GEMM_ZX, 1, s);
      if (p.fast_gemm) {
        if (ldx != p.n_in) {
          if (!x_padded) HIPCHK(launch_pad_rows(x, ws + p.ws_xpad, (long)(T * B), p.n_in, ldx, s));
          g.A = ws + p.ws_xpad;
        }
        g.K = ldx; g.lda = ldx;
        g.k_phys_rows = p.n_in;          // (W_x as it lies in memory)
        if (p.zx_nn) { g.parts = (float*)(ws + p.ws_parts); g.parts_bytes = p.parts_bytes; }
        const bool fast = p.zx_nn ? gemm_tile_ok(g) : gemm_nn_ok(g);
        if (!fast) { g.K = p.n_in; g.k_phys_rows = 0; g.parts = nullptr; }      // (operands past 2 GiB: the generic kernel, which knows no padding)
        if (seq_lens && fast) {
          // only real frames are projected: row r of the product is frame fidx[r]; the pre-activations of padded
          // frames stay unwritten and are never read
          int* fidx = (int*)(ws + p.ws_fidx);
          int* count = (int*)(ws + p.ws_count);
          if (!frames_mapped) HIPCHK(launch_frame_map(seq_lens, p.T, p.B, fidx, count, s));
          g.a_rows = fidx; g.c_rows = fidx; g.a_phys_rows = g.M; g.m_dev = count;
        }
      } else if (!p.bf16) {              // float storage: the same padding, the same selection of real frames
        g.parts = (float*)(ws + p.ws_parts); g.parts_bytes = p.parts_bytes;
        if (p.n_in8 != p.n_in) {
          const GemmArgs gp = padded_float(g);
          if (gemm_float_ok(gp)) {
            if (!x_padded) HIPCHK(launch_pad_rows(x, ws + p.ws_xpad, (long)(T * B), 2 * p.n_in, 2 * p.n_in8, s));
            g = gp;
          }
        }
        if (seq_lens) {
          int* fidx = (int*)(ws + p.ws_fidx);
          int* count = (int*)(ws + p.ws_count);
          if (!frames_mapped) HIPCHK(launch_frame_map(seq_lens, p.T, p.B, fidx, count, s));
          g.a_rows = fidx; g.c_rows = fidx; g.a_phys_rows = g.M; g.m_dev = count;
        }
      }
      HIPCHK(launch_gemm(g, s));
    }
    return LSTM_OK;
  };
  if (p.small) {                         // a narrow layer: projection and loop, nothing to set up
    if (p.zx_tiny) {
      Phase ph(LSTM_PHASE_GEMM_ZX, 1, s);
      TinyGroup g = {};
      g.p[g.count++] = tiny_zx(p, x, W_x, b, gates, gates_stride);
      HIPCHK(launch_gemm_tiny(g, p.bf16, nullptr, nullptr, s));
    } else if ((rc = project())) return rc;
    SmallFwdArgs a = {};
    a.lens = seq_lens; a.B = p.B; a.n = p.n; a.T = p.T; a.ndir = p.D; a.write_gates = infer ? 0 : 1; a.sync = (unsigned*)(ws + p.ws_sync);
    for (size_t d = 0; d < D; ++d) {
      SmallFwdDir& fd = a.d[d];
      fd.W = (const char*)W_h + d * n * 4 * n * p.esz;
      fd.gates = gates + d * gates_stride;
      fd.h0 = h0 ? (const float*)h0 + d * B * n : nullptr; fd.c0 = c0 ? (const float*)c0 + d * B * n : nullptr;
      fd.hT = hT ? (float*)hT + d * B * n : nullptr; fd.cT = cT ? (float*)cT + d * B * n : nullptr;
      fd.y = (char*)y + d * n * p.esz; fd.ldy = (long)(D * n);
      fd.cs = c ? (float*)c + d * T * B * n : nullptr;
      fd.hprev = infer ? nullptr : rs + d * p.res_dir_stride + p.res_hprev; fd.ldh = p.ldh;
      fd.rev = bidir ? d == 1 : desc->direction == -1;
    }
    Phase ph(LSTM_PHASE_LOOP_FWD, 1, s);
    HIPCHK(launch_small_fwd(a, p.bf16, s));
    return LSTM_OK;
  }
  if (p.blocks && loop_block_pays(p.T, p.B, p.n, p.D, (desc->flags & LSTM_FLAG_PLAIN_LAUNCH) != 0, false) && loop_block_fits(p.B, p.n, (long)(D * n))) {    // a wide layer: projection, then a launch per direction and 32 rows
    // Until a row's first frame every column of the grid reads its h0 from memory, and the columns do not end together: a state in
    // place (hT over h0) is read from a copy.
    if (bytes_overlap(h0, state_bytes, hT, state_bytes) || bytes_overlap(h0, state_bytes, cT, state_bytes)) {
      HIPCHK(launch_copy(hstate, h0, state_bytes, s));
      h0 = hstate;
    }
    if ((rc = project())) return rc;
    hipError_t e = hipSuccess;
    for (size_t d = 0; d < D && e == hipSuccess; ++d) {
      BlockFwdArgs a = {};
      a.W = ws + p.ws_blocks; a.gates = gates + d * gates_stride;
      a.h0 = h0 ? (const float*)h0 + d * B * n : nullptr; a.c0 = c0 ? (const float*)c0 + d * B * n : nullptr;
      a.hT = hT ? (float*)hT + d * B * n : nullptr; a.cT = cT ? (float*)cT + d * B * n : nullptr;
      a.y = (char*)y + d * n * p.esz; a.ldy = (long)(D * n);
      a.cs = c ? (float*)c + d * T * B * n : nullptr;
      a.hprev = infer ? nullptr : rs + d * p.res_dir_stride + p.res_hprev; a.ldh = p.ldh;
      a.rev = bidir ? d == 1 : desc->direction == -1;
      a.lens = seq_lens; a.B = p.B; a.n = p.n; a.T = p.T; a.write_gates = infer ? 0 : 1;
      a.ring = ws + p.ws_blocks + loop_block_wh_bytes(p.n); a.ring_bytes = loop_block_ring_bytes(p.n);
      a.sync = (unsigned*)(ws + p.ws_sync); a.xcc = a.sync + 64; a.spin_limit = kSpinLimit;
      a.plain_launch = (desc->flags & LSTM_FLAG_PLAIN_LAUNCH) != 0; a.first = d == 0;
      {
        Phase ph(LSTM_PHASE_PREP, 1, s);
        HIPCHK(launch_pack_blocks((const char*)W_h + d * n * 4 * n * p.esz, a, s));
      }
      Phase ph(LSTM_PHASE_LOOP_FWD, 2, s);                 // (counted with the clearing, as backward, though that rides in the launch before)
      e = launch_block_fwd(a, s);
      if (e != hipSuccess && (d > 0 || e != hipErrorCooperativeLaunchTooLarge)) return LSTM_ERR_HIP;
    }
    if (e == hipSuccess) return LSTM_OK;
    (void)hipGetLastError();               // refused before anything ran: the per-step path
  }
  const PackRows rows = pack_rows(p, ws, seq_lens, false, desc);
  const bool paired = rows.slots > 0 || persist_fwd_rows(p.B, p.n, p.D) == 8;    // (how the bf16 single-launch kernel wants W_h)
  const GemmArgs zx = projection();
  // Only without a reserve: sums come in another order here, and in training a last place decides which frame a maximum over time sends its gradient to
  // (six layers pooled by 8, 200 - 1500 frames: gradients moved by 2.7 %).
  const bool w_rows = infer && p.bf16 && !(desc->flags & LSTM_FLAG_PER_STEP) && T >= 2 && p.nkc_ll_f <= kLLMaxNkcFwd && rows.slots == 0 && paired && persist_fwd_w_rows(p.B, p.n, p.D);
  projected = w_rows && few_zx_ok(zx);
  // single-launch path: bf16 storage, at least two steps, register budget of the kernel
  bool use_ll = p.bf16 && !(desc->flags & LSTM_FLAG_PER_STEP) && T >= 2 && p.nkc_ll_f <= kLLMaxNkcFwd;
  // what the per-step kernels work on (also what a single-launch path that does not start falls back to)
  auto pack_w = [&]() -> int {
    Phase ph(LSTM_PHASE_PREP, 1, s);
    HIPCHK(launch_pack_wh_fwd(W_h, (uint4*)(ws + p.ws_Wf), p.n, p.nkc_f, p.D, p.bf16, s));
    return LSTM_OK;
  };
  auto state_in = [&]() -> int {
    Phase ph(LSTM_PHASE_PREP, 3, s);
    if (h0) HIPCHK(launch_copy(hstate, h0, state_bytes, s)); else HIPCHK(launch_fill_zero(hstate, state_bytes, s));
    if (c0) HIPCHK(launch_copy(cstate, c0, state_bytes, s)); else HIPCHK(launch_fill_zero(cstate, state_bytes, s));
    if (T > 0)
      HIPCHK(launch_pack_state(hstate, (uint4*)(ws + p.ws_hfrag0), (uint4*)(ws + p.ws_hfrag1), p.B, p.n, p.nkc_f, p.nrt, p.D, p.bf16, s));
    return LSTM_OK;
  };
  // The initial state does not travel through the exchange rings (what does must keep |h| <= 1): its product with W_h goes into the
  // pre-activations of every row's first frame, and the kernels start from zeros in the ring.  (B rows, but W_h is read once
  // for all of them: a kernel with a thread per column and row took 270 us for 32 rows of 1024 units.)
  auto h0_term = [&]() -> int {            // (its operands by the set-up launch)
    Phase ph(LSTM_PHASE_PREP, p.D, s);
    int* rows = (int*)(ws + p.ws_h0rows);
    for (size_t d = 0; d < D; ++d) {
      GemmArgs g = {};
      g.A = ws + p.ws_h0 + d * B * p.ldh * p.esz; g.B = (const char*)W_h + d * n * 4 * n * p.esz; g.C = gates + d * gates_stride;
      g.M = p.B; g.N = 4 * p.n; g.K = (int)p.ldh; g.lda = p.ldh; g.ldb = 4 * n; g.ldc = 4 * n; g.nz = 1; g.nseg = 1;
      g.a_kcontig = true; g.in_bf16 = p.bf16; g.accumulate = 1; g.c_rows = rows + d * B; g.k_phys_rows = p.n;
      g.parts = (float*)(ws + p.ws_parts); g.parts_bytes = p.parts_bytes;
      if (!(p.bf16 ? gemm_tile_ok(g) : gemm_float_ok(g))) { g.K = p.n; g.k_phys_rows = 0; g.parts = nullptr; }
      HIPCHK(launch_gemm(g, s));
    }
    return LSTM_OK;
  };
  bool done = false;
  auto set_dirs = [&](PFwdArgs& pa, const char* Wf, size_t wf_dir, size_t frag_dir) {
    pa.lens = seq_lens; pa.B = p.B; pa.n = p.n; pa.T = p.T; pa.ndir = p.D; pa.write_gates = infer ? 0 : 1;
    pa.plain_launch = (desc->flags & LSTM_FLAG_PLAIN_LAUNCH) != 0;
    pa.sync = (unsigned*)(ws + p.ws_sync); pa.spin_limit = kSpinLimit;
    pa.xcc = (unsigned*)(ws + p.ws_sync) + 64 + 2 * (size_t)p.nrt;
    for (size_t d = 0; d < D; ++d) {
      PFwdDir& fd = pa.d[d];
      fd.Wf = (const uint4*)(Wf + d * wf_dir);
      fd.Wzero = (const uint4*)(ws + p.ws_Wf + p.Wf_bytes);
      fd.ring0 = (uint4*)(ws + p.ws_hfrag0 + d * frag_dir);
      fd.ring1 = (uint4*)(ws + p.ws_hfrag1 + d * frag_dir);
      fd.gates = gates + d * gates_stride;
      fd.h0 = h0 ? (const float*)h0 + d * B * n : nullptr; fd.c0 = c0 ? (const float*)c0 + d * B * n : nullptr;
      fd.hT = hT ? (float*)hT + d * B * n : nullptr; fd.cT = cT ? (float*)cT + d * B * n : nullptr;
      fd.y = (char*)y + d * n * p.esz;
      fd.ldy = (long)(D * n);
      fd.cs = c ? (float*)c + d * T * B * n : nullptr;
      fd.hprev = infer ? nullptr : rs + d * p.res_dir_stride + p.res_hprev;
      fd.ldh = p.ldh;
      fd.rev = bidir ? d == 1 : desc->direction == -1;
      fd.tab = fd.rev ? rows.down : rows.up;
    }
  };
  PFwdArgs pa = {};                      // the single-launch kernels' arguments, if one of them takes this problem
  if (use_ll) {
    pa.nkc = p.nkc_ll_f; pa.slots = rows.slots; pa.tab_steps = rows.tab_steps; pa.steps = rows.steps;
    pa.w_rows = w_rows;
    if (w_rows) set_dirs(pa, (const char*)W_h, n * 4 * n * p.esz, (size_t)p.nrt * p.nkc_ll_f * 1024);
    else set_dirs(pa, ws + p.ws_Wf, ll_wf_bytes(p.n, p.nkc_ll_f), (size_t)p.nrt * p.nkc_ll_f * 1024);
  } else {
    pa.nkc = p.nkc_f;                    // (float storage: the per-step kernels' packed W_h and h buffers)
    set_dirs(pa, ws + p.ws_Wf, (size_t)p.ntile_f * 2 * p.nkc_f * 1024, (size_t)p.nrt * p.nkc_f * 1024);
  }
  const bool use_ll32 = !p.bf16 && !(desc->flags & LSTM_FLAG_PER_STEP) && T >= 2 && persist_fwd_f32_fits(pa) &&
                        persist_f32_pays(p.T, p.B, p.n, p.D, seq_lens != nullptr, pa.plain_launch, false);
  const bool single = use_ll ? persist_fwd_fits(pa) : use_ll32;
  SetUpCopies copies = {};
  if (T > 0 && !projected && ldx != p.n_in && (p.bf16 || gemm_float_ok(padded_float(zx)))) {
    const int words = p.bf16 ? 1 : 2;    // (16-bit ones)
    copies.x = x; copies.xpad = ws + p.ws_xpad; copies.x_rows = (long)(T * B); copies.x_cols = words * p.n_in; copies.x_ld = words * ldx;
  }
  if (T > 0 && single && h0) {
    copies.h0 = (const float*)h0; copies.out = ws + p.ws_h0; copies.row = (int*)(ws + p.ws_h0rows); copies.ld = (int)p.ldh;
    copies.rev0 = pa.d[0].rev; copies.rev1 = pa.d[D - 1].rev;
    copies.lens = seq_lens; copies.T = p.T; copies.B = p.B; copies.n = p.n; copies.ndir = p.D;
  }
  {
    Phase ph(projected ? LSTM_PHASE_GEMM_ZX : LSTM_PHASE_PREP, projected ? 1 : 5, s);
    ZeroRegions z;
    z.add(ws + p.ws_sync, p.sync_bytes);
    if (use_ll)
      z.add(ws + p.ws_Wf + p.Wf_bytes, 1024);              // the chunk of zeros behind the packed W_h (single-launch path)
    // (on the single-launch paths the fills, the packed W_h and the initial ring are one launch)
    if (use_ll) {
      FrameMapArgs fm = {};
      if (p.fast_gemm && seq_lens && !projected) {   // the input projection below goes over the real frames
        fm = {seq_lens, p.T, p.B, (int*)(ws + p.ws_fidx), (int*)(ws + p.ws_count)};
        frames_mapped = true;
      }
      HIPCHK(launch_prep_fwd_ll(z, W_h, w_rows ? nullptr : (uint4*)(ws + p.ws_Wf), p.n, p.nkc_ll_f, p.D, paired, (uint4*)(ws + p.ws_hfrag0), (uint4*)(ws + p.ws_hfrag1),
                                p.nrt, fm, rows, copies, projected ? &zx : nullptr, s));
    } else if (use_ll32) {
      FrameMapArgs fm = {};
      if (seq_lens) {
        fm = {seq_lens, p.T, p.B, (int*)(ws + p.ws_fidx), (int*)(ws + p.ws_count)};
        frames_mapped = true;
      }
      HIPCHK(launch_prep_fwd_f32(z, W_h, ws + p.ws_Wf, pa, fm, copies, s));
    } else HIPCHK(launch_fill_zero_many(z, s));
    x_padded = copies.x && (use_ll || use_ll32);
  }
  if (T > 0 && !single && (rc = pack_w())) return rc;
  if (!single && (rc = state_in())) return rc;
  if (T > 0) {
    if ((rc = project())) return rc;
    if (single) {
      if (h0 && (rc = h0_term())) return rc;
      // The fill behind rows one behind the other gives padded frames of a reversed direction the state that the call began with, and by then the
      // loop has stored cT: a state in place (cT over c0) is read from a copy.
      const float* c0_fill = (const float*)c0;
      if (pa.slots > 0 && c && (pa.d[0].rev || pa.d[D - 1].rev) && bytes_overlap(c0, state_bytes, cT, state_bytes)) {
        Phase ph(LSTM_PHASE_PREP, 1, s);
        HIPCHK(launch_copy(cstate, c0, state_bytes, s));
        c0_fill = cstate;
      }
      hipError_t e;
      {
        Phase ph(LSTM_PHASE_LOOP_FWD, pa.slots > 0 ? 2 : 1, s);
        e = use_ll ? launch_persist_fwd(pa, s) : launch_persist_fwd_f32(pa, s);
        if (e == hipSuccess && pa.slots > 0) {
          float* cs[2] = {pa.d[0].cs, pa.d[D - 1].cs};
          const float* cz[2] = {c0_fill, c0_fill ? c0_fill + (D - 1) * B * n : nullptr};
          const int rev[2] = {pa.d[0].rev, pa.d[D - 1].rev};
          HIPCHK(launch_fill_padded(seq_lens, rows.steps, p.T, p.B, p.n, p.D, y, cs, cz, rev, s));
        }
      }
      if (e == hipErrorCooperativeLaunchTooLarge && h0) e = hipErrorLaunchFailure;   // the pre-activations are no longer what the per-step path expects
      if (e == hipSuccess) done = true;
      else if (e == hipErrorCooperativeLaunchTooLarge) {   // nothing was launched (does not fit on the device all at once): one launch per step
        (void)hipGetLastError();
        if (use_ll && (rc = pack_w())) return rc;
        if ((rc = state_in())) return rc;
      } else {                                      // a later batch slab failed after earlier ones ran: no second attempt on advanced state
        (void)hipGetLastError();
        return LSTM_ERR_HIP;
      }
    }
    if (!done) {
    Phase ph(LSTM_PHASE_LOOP_FWD, (long)T, s);
    FwdArgs a = {};
    a.lens = seq_lens; a.B = p.B; a.n = p.n; a.nkc = p.nkc_f; a.T = p.T; a.ndir = p.D; a.write_gates = infer ? 0 : 1;
    const size_t frag_dir = (size_t)p.nrt * p.nkc_f * 1024;
    for (size_t tau = 0; tau < T; ++tau) {
      for (size_t d = 0; d < D; ++d) {
        const bool rev = bidir ? d == 1 : desc->direction == -1;
        const size_t t = rev ? T - 1 - tau : tau;
        FwdDir& fd = a.d[d];
        fd.Wf = (const uint4*)(ws + p.ws_Wf + d * (size_t)p.ntile_f * 2 * p.nkc_f * 1024);
        fd.hin = (const uint4*)(ws + ((tau & 1) ? p.ws_hfrag1 : p.ws_hfrag0) + d * frag_dir);
        fd.hout = ws + ((tau & 1) ? p.ws_hfrag0 : p.ws_hfrag1) + d * frag_dir;
        fd.gates = gates + d * gates_stride + t * B * 4 * n;
        fd.hstate = hstate + d * B * n;
        fd.cstate = cstate + d * B * n;
        fd.y = (char*)y + (t * B * D * n + d * n) * p.esz;
        fd.ldy = (long)(D * n);
        fd.cs = c ? (float*)c + (d * T + t) * B * n : nullptr;
        fd.hprev = infer ? nullptr : rs + d * p.res_dir_stride + p.res_hprev + t * B * p.ldh * p.esz;
        fd.ldh = p.ldh;
        fd.t = (int)t;
      }
      HIPCHK(launch_step_fwd(a, p.bf16, s));
    }
    }
  }
  if (done) return LSTM_OK;
  Phase ph(LSTM_PHASE_PREP, 2, s);
  if (hT) HIPCHK(launch_copy(hT, hstate, state_bytes, s));
  if (cT) HIPCHK(launch_copy(cT, cstate, state_bytes, s));
  return LSTM_OK;
}

int run_bwd(const lstm_desc* desc, int bidir, const void* x, const void* W_x, const void* W_h, const void* h0,
            const void* c0, const int32_t* seq_lens, const void* y, const void* c, const void* reserve, const void* dy,
            const void* dhT, const void* dcT, void* dx, void* dW_x, void* dW_h, void* db, void* dh0, void* dc0,
            void* workspace, void* stream) {
  Plan p;
  int rc = call_plan(desc, bidir, &p);
  if (rc) return rc;
  if (!bidir && desc->direction != 1 && desc->direction != -1) return LSTM_ERR_DIRECTION;
  if (desc->flags & LSTM_FLAG_INFERENCE) return LSTM_ERR_UNSUPPORTED;
  if (!x || !W_x || !W_h || !c || !reserve || !dy || !dW_x || !dW_h || !db || !workspace) return LSTM_ERR_NULL;
  const void* ptrs[] = {x, W_x, W_h, h0, c0, seq_lens, y, c, reserve, dy, dhT, dcT, dx, dW_x, dW_h, db, dh0, dc0, workspace};
  for (const void* q : ptrs) if (misaligned(q)) return LSTM_ERR_ALIGN;
  if (desc->workspace_bytes < p.workspace_bytes || desc->reserve_bytes < p.reserve_bytes) return LSTM_ERR_SIZE;
  if ((rc = check_device())) return rc;

  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)(((uintptr_t)workspace + kAlign - 1) / kAlign * kAlign);
  const char* rs = (const char*)(((uintptr_t)reserve + kAlign - 1) / kAlign * kAlign);
  const size_t n = p.n, B = p.B, D = p.D, T = p.T, n_in = p.n_in;
  const int acc = (desc->flags & LSTM_FLAG_ACCUMULATE) ? 1 : 0;
  float* Dh = (float*)(ws + p.ws_Dh);
  float* Dc = (float*)(ws + p.ws_Dc);
  const size_t state_bytes = D * B * n * 4;
  if (B > 0 && T == 0) HIPCHK(launch_fill_zero(ws + p.ws_sync, p.sync_bytes, s));
  if (B == 0 || T == 0) {          // no frames: parameter gradients are zero, state gradients pass through
    if (!acc) {
      HIPCHK(launch_fill_zero(dW_x, D * n_in * 4 * n * 4, s));
      HIPCHK(launch_fill_zero(dW_h, D * n * 4 * n * 4, s));
      HIPCHK(launch_fill_zero(db, D * 4 * n * 4, s));
    }
    if (B > 0) {
      if (dh0) { if (dhT) HIPCHK(launch_copy(dh0, dhT, state_bytes, s)); else HIPCHK(launch_fill_zero(dh0, state_bytes, s)); }
      if (dc0) { if (dcT) HIPCHK(launch_copy(dc0, dcT, state_bytes, s)); else HIPCHK(launch_fill_zero(dc0, state_bytes, s)); }
    }
    return LSTM_OK;
  }
  // With sequence lengths given, the products behind the loop run over the real frames only (about two thirds of T*B for
  // the length mix of speech batches): frames are numbered once, row-indexed products gather / scatter through
  // that numbering and the transposed operands of the weight gradients are packed by it.
  const int TB = (int)(T * B);
  const bool compact = (p.fast_gemm || !p.bf16) && seq_lens && TB > 0;
  char* DZ = ws + p.ws_DZ;
  bool dx_cleared = false, frames_mapped = false, x_padded = false;      // done by a set-up launch of the loop
  int db_slices = 0;                                   // slices of the bias gradient that the loop leaves in ws_colsum (0: none)
  TinyGroup tiny = {};
  if (p.dw_tiny) tiny = tiny_bwd(p, x, W_x, rs + p.res_hprev, DZ, seq_lens, dx, dW_x, dW_h, acc);
  bool db_done = false;

  auto narrow_loop = [&]() -> int {
    SmallBwdArgs a = {};
    const int slices = cdiv((long)B, 4);
    a.lens = seq_lens; a.B = p.B; a.n = p.n; a.T = p.T; a.ndir = p.D; a.accumulate = acc; a.sync = (unsigned*)(ws + p.ws_sync);
    if (p.dw_tiny) { a.counters = (unsigned*)(ws + p.ws_tiny_cnt); a.ncounters = tiny_counters(tiny); }
    for (size_t d = 0; d < D; ++d) {
      SmallBwdDir& bd = a.d[d];
      bd.W = (const char*)W_h + d * n * 4 * n * p.esz;
      bd.gates = (const float*)(rs + d * p.res_dir_stride + p.res_gates);
      bd.cs = (const float*)c + d * T * B * n;
      bd.c0 = c0 ? (const float*)c0 + d * B * n : nullptr;
      bd.dy = (const char*)dy + d * n * p.esz; bd.lddy = (long)(D * n);
      bd.DZ = DZ + d * p.DZ_dir_elems * p.esz;
      bd.dhT = dhT ? (const float*)dhT + d * B * n : nullptr; bd.dcT = dcT ? (const float*)dcT + d * B * n : nullptr;
      bd.dh0 = dh0 ? (float*)dh0 + d * B * n : nullptr; bd.dc0 = dc0 ? (float*)dc0 + d * B * n : nullptr;
      bd.db = slices <= kColsumSlices ? (float*)db + d * 4 * n : nullptr;
      bd.dbpart = (float*)(ws + p.ws_colsum) + d * kColsumSlices * 4 * n;
      bd.rev = bidir ? d == 1 : desc->direction == -1;
    }
    db_done = slices == 1;
    db_slices = slices <= kColsumSlices ? slices : 0;
    Phase ph(LSTM_PHASE_LOOP_BWD, 1, s);
    HIPCHK(launch_small_bwd(a, p.bf16, s));
    return LSTM_OK;
  };

  auto split_loop = [&]() -> int {
    // single-launch path: bf16 storage, at least two steps, and the kernel fits the device
    PBwdArgs pa = {};
    pa.lens = seq_lens; pa.B = p.B; pa.n = p.n; pa.T = p.T; pa.ndir = p.D;
    pa.plain_launch = (desc->flags & LSTM_FLAG_PLAIN_LAUNCH) != 0;
    pa.sync = (unsigned*)(ws + p.ws_sync); pa.spin_limit = kSpinLimit;
    pa.xcc = (unsigned*)(ws + p.ws_sync) + 64 + 2 * (size_t)p.nrt;
    for (size_t d = 0; d < D; ++d) pa.d[d].lddy = (long)(D * n);       // (the check looks at the frame sizes)
    const bool use_ll = p.bf16 && !(desc->flags & LSTM_FLAG_PER_STEP) && T >= 2 && persist_bwd_fits(pa);
    PackRows rows = {};
    if (use_ll && compact) rows = pack_rows(p, ws, seq_lens, true, desc);
    pa.slots = rows.slots; pa.tab_steps = rows.tab_steps; pa.steps = rows.steps;
    const bool eights = persist_bwd_rows(p.B, p.n, p.D) == 8;
    const int wb_nct = eights && rows.slots == 0 ? bwdp8_nct(p.n) : bwdp_nct(p.n);
    const bool use_ll32 = !p.bf16 && !(desc->flags & LSTM_FLAG_PER_STEP) && T >= 2 && p.n <= 1024 && p.B <= 256 &&
                          persist_bwd_f32_fits(pa) && persist_f32_pays(p.T, p.B, p.n, p.D, seq_lens != nullptr, pa.plain_launch, true);
    {
      Phase ph(LSTM_PHASE_PREP, 5, s);
      ZeroRegions z;
      z.add(ws + p.ws_sync, p.sync_bytes);
      z.add(ws + p.ws_dzfrag0, p.dzfrag_bytes);
      z.add(ws + p.ws_dzfrag1, p.dzfrag_bytes);
      if (2 * p.nrt <= kColsumSlices) z.add(ws + p.ws_colsum, D * kColsumSlices * 4 * n * 4);   // bias-gradient slices of row groups the grid lacks
      // (the single-launch paths clear and pack W_h^T in one launch)
      if (use_ll || use_ll32) {
        FrameMapArgs fm = {};
        if (compact) {
          fm = {seq_lens, p.T, p.B, (int*)(ws + p.ws_fidx), (int*)(ws + p.ws_count)};
          frames_mapped = true;
        }
        if (compact && dx && ((size_t)TB * n_in * p.esz) % 4 == 0) {   // dX is scattered to the real frames' rows: the padded frames' rows are cleared here
          z.add(dx, (size_t)TB * n_in * p.esz);
          dx_cleared = true;
        }
        SetUpCopies copies = {};
        if (p.n_in8 != p.n_in && (p.fast_gemm || !p.bf16)) {               // x in rows of whole 16 bytes, for dW_x
          const int words = p.bf16 ? 1 : 2;
          copies.x = x; copies.xpad = ws + p.ws_xpad; copies.x_rows = TB; copies.x_cols = words * p.n_in; copies.x_ld = words * p.n_in8;
          x_padded = true;
        }
        if (use_ll32) HIPCHK(launch_prep_bwd_f32(z, W_h, ws + p.ws_Wb, p.n, p.D, fm, copies, s));
        else HIPCHK(launch_prep_bwd_ll(z, W_h, (uint4*)(ws + p.ws_Wb), p.n, p.D, rows.slots > 0 || eights, wb_nct, fm, rows, copies, s));
      } else HIPCHK(launch_fill_zero_many(z, s));
    }
    if (!use_ll && !use_ll32) {
      Phase ph(LSTM_PHASE_PREP, 1, s);
      HIPCHK(launch_pack_wh_bwd(W_h, (uint4*)(ws + p.ws_Wb), p.n, p.nkc_b, p.D, p.bf16, s));
    }

    const size_t frag_dir = (size_t)p.nrt * p.nkc_b * 1024;
    bool done = false;
    const bool db_in_loop = (use_ll || use_ll32) && 2 * p.nrt <= kColsumSlices;   // the single-launch kernels also sum the bias gradient
    if (use_ll || use_ll32) {
      const size_t ring_dir = use_ll ? bwdp_ring_bytes(p.B, p.n) : bwd_f32_ring_bytes(p.B, p.n);
      const size_t wb_dir = use_ll ? bwdp_wh_bytes(p.n, wb_nct) : bwd_f32_wh_bytes(p.n);
      for (size_t d = 0; d < D; ++d) {
        PBwdDir& bd = pa.d[d];
        bd.Wb = (const uint4*)(ws + p.ws_Wb + d * wb_dir);
        bd.ring0 = (uint4*)(ws + p.ws_dzfrag0 + d * ring_dir);
        bd.ring1 = (uint4*)(ws + p.ws_dzfrag1 + d * ring_dir);
        bd.wide = use_ll32 ? (uint4*)(ws + p.ws_dzwide + d * ring_dir) : nullptr;
        bd.gates = (const float*)(rs + d * p.res_dir_stride + p.res_gates);
        bd.cs = (const float*)c + d * T * B * n;
        bd.c0 = c0 ? (const float*)c0 + d * B * n : nullptr;
        bd.dy = (const char*)dy + d * n * p.esz;
        bd.lddy = (long)(D * n);
        bd.DZ = DZ + d * p.DZ_dir_elems * p.esz;
        bd.dhT = dhT ? (const float*)dhT + d * B * n : nullptr; bd.dcT = dcT ? (const float*)dcT + d * B * n : nullptr;
        bd.dh0 = dh0 ? (float*)dh0 + d * B * n : nullptr; bd.dc0 = dc0 ? (float*)dc0 + d * B * n : nullptr;
        bd.dbpart = db_in_loop ? (float*)(ws + p.ws_colsum) + d * kColsumSlices * 4 * n : nullptr;
        bd.rev = bidir ? d == 1 : desc->direction == -1;
        bd.tab = bd.rev ? rows.up : rows.down;
      }
      hipError_t e;
      {
        Phase ph(LSTM_PHASE_LOOP_BWD, 1, s);
        e = use_ll ? launch_persist_bwd(pa, s) : launch_persist_bwd_f32(pa, s);
      }
      if (e == hipSuccess) {
        done = true;
        if (db_in_loop) db_slices = 2 * p.nrt;
      }
      else if (e != hipErrorCooperativeLaunchTooLarge) {   // a later batch slab failed after earlier ones ran
        (void)hipGetLastError();
        return LSTM_ERR_HIP;
      } else {
        (void)hipGetLastError();
        Phase ph(LSTM_PHASE_PREP, 1, s);
        HIPCHK(launch_pack_wh_bwd(W_h, (uint4*)(ws + p.ws_Wb), p.n, p.nkc_b, p.D, p.bf16, s));
      }
    }
    BwdArgs a = {};
    a.lens = seq_lens; a.B = p.B; a.n = p.n; a.nkc = p.nkc_b; a.T = p.T; a.ndir = p.D;
    if (done) return LSTM_OK;
    {
      Phase ph(LSTM_PHASE_PREP, 2, s);
      if (dhT) HIPCHK(launch_copy(Dh, dhT, state_bytes, s)); else HIPCHK(launch_fill_zero(Dh, state_bytes, s));
      if (dcT) HIPCHK(launch_copy(Dc, dcT, state_bytes, s)); else HIPCHK(launch_fill_zero(Dc, state_bytes, s));
    }
    {
    Phase ph(LSTM_PHASE_LOOP_BWD, (long)T + 1, s);
    for (long tau = (long)T - 1; tau >= -1; --tau) {
      a.do_matmul = tau < (long)T - 1;
      a.do_pointwise = tau >= 0;
      for (size_t d = 0; d < D; ++d) {
        const bool rev = bidir ? d == 1 : desc->direction == -1;
        const long t = rev ? (long)T - 1 - tau : tau;            // frame of this step (out of range when tau == -1)
        const long t_next = rev ? t - 1 : t + 1;                 // frame of the previous backward step
        BwdDir& bd = a.d[d];
        bd.Wb = (const uint4*)(ws + p.ws_Wb + d * (size_t)p.ntile_b * p.nkc_b * 1024);
        bd.dzin = (const uint4*)(ws + (((tau + 1) & 1) ? p.ws_dzfrag1 : p.ws_dzfrag0) + d * frag_dir);
        bd.dzout = ws + ((tau & 1) ? p.ws_dzfrag1 : p.ws_dzfrag0) + d * frag_dir;
        bd.Dh = Dh + d * B * n;
        bd.Dc = Dc + d * B * n;
        bd.t = (int)t; bd.t_next = (int)t_next;
        if (tau >= 0) {
          const float* cs = (const float*)c + d * T * B * n;
          const long tp = rev ? t + 1 : t - 1;                   // frame processed just before t in the forward pass
          bd.gates = (const float*)(rs + d * p.res_dir_stride + p.res_gates) + t * B * 4 * n;
          bd.cs = cs + t * B * n;
          bd.cprev = (tp >= 0 && tp < (long)T) ? cs + tp * B * n : (c0 ? (const float*)c0 + d * B * n : nullptr);
          bd.dy = (const char*)dy + (t * B * D * n + d * n) * p.esz;
          bd.lddy = (long)(D * n);
          bd.DZ = DZ + (d * p.DZ_dir_elems + t * B * 4 * n) * p.esz;
        }
      }
      HIPCHK(launch_step_bwd(a, p.bf16, s));
    }
    }
    {
      Phase ph(LSTM_PHASE_PREP, 2, s);
      if (dh0) HIPCHK(launch_copy(dh0, Dh, state_bytes, s));
      if (dc0) HIPCHK(launch_copy(dc0, Dc, state_bytes, s));
    }
    return LSTM_OK;
  };
  auto block_loop = [&]() -> int {
    const int slices = 4 * cdiv((long)B, 16);
    for (size_t d = 0; d < D; ++d) {
      BlockBwdArgs a = {};
      a.W = (const char*)W_h + d * n * 4 * n * p.esz;
      a.gates = (const float*)(rs + d * p.res_dir_stride + p.res_gates);
      a.cs = (const float*)c + d * T * B * n;
      a.c0 = c0 ? (const float*)c0 + d * B * n : nullptr;
      a.dhT = dhT ? (const float*)dhT + d * B * n : nullptr; a.dcT = dcT ? (const float*)dcT + d * B * n : nullptr;
      a.dh0 = dh0 ? (float*)dh0 + d * B * n : nullptr; a.dc0 = dc0 ? (float*)dc0 + d * B * n : nullptr;
      a.dy = (const char*)dy + d * n * p.esz; a.lddy = (long)(D * n);
      a.DZ = DZ + d * p.DZ_dir_elems * p.esz;
      a.dbpart = slices <= kColsumSlices ? (float*)(ws + p.ws_colsum) + d * kColsumSlices * 4 * n : nullptr;
      a.rev = bidir ? d == 1 : desc->direction == -1;
      a.lens = seq_lens; a.B = p.B; a.n = p.n; a.T = p.T;
      a.ring = ws + p.ws_blocks + loop_block_wh_bytes(p.n); a.ring_bytes = loop_block_ring_bytes_bwd(p.n);
      a.sync = (unsigned*)(ws + p.ws_sync); a.xcc = a.sync + 64; a.spin_limit = kSpinLimit;
      a.plain_launch = (desc->flags & LSTM_FLAG_PLAIN_LAUNCH) != 0; a.first = d == 0;
      Phase ph(LSTM_PHASE_LOOP_BWD, 2, s);
      const hipError_t e = launch_block_bwd(a, s);
      if (e == hipErrorCooperativeLaunchTooLarge && d == 0) {      // refused before anything ran
        (void)hipGetLastError();
        return split_loop();
      }
      HIPCHK(e);
    }
    db_slices = slices <= kColsumSlices ? slices : 0;
    return LSTM_OK;
  };

  const bool blocks = p.blocks && loop_block_pays(p.T, p.B, p.n, p.D, (desc->flags & LSTM_FLAG_PLAIN_LAUNCH) != 0, true) &&
                      loop_block_fits(p.B, p.n, (long)(D * n));
  if ((rc = p.small ? narrow_loop() : blocks ? block_loop() : split_loop())) return rc;

  int* fidx = (int*)(ws + p.ws_fidx);
  int* count = (int*)(ws + p.ws_count);
  if (compact && !frames_mapped && !p.dw_tiny) {
    Phase ph(LSTM_PHASE_PREP, 1, s);
    HIPCHK(launch_frame_map(seq_lens, p.T, p.B, fidx, count, s));
  }
  SumList sums;                        // what the products' K ranges and the loop's bias-gradient slices still have to be added to
  auto parts_of = [&](GemmArgs& g) { g.parts = (float*)(ws + p.ws_parts + sums.used); g.parts_bytes = p.parts_bytes - sums.used; g.sums = &sums; };
  auto products = [&]() -> int {
    GemmArgs gd = {};                // dX = sum over directions of DZ W_x^T
    bool fill_dx = false, parts_dx = false;
    if (dx) {
      GemmArgs& g = gd;
      g.A = DZ; g.B = W_x; g.C = dx;
      g.M = TB; g.N = p.n_in; g.K = 4 * p.n;
      g.lda = 4 * n; g.ldb = 4 * n; g.ldc = n_in; g.nz = 1;
      g.nseg = p.D; g.sAseg = (long)p.DZ_dir_elems; g.sBseg = (long)(n_in * 4 * n); g.frames = true;
      g.a_kcontig = true; g.b_kcontig = true; g.in_bf16 = p.bf16; g.out_bf16 = p.bf16;
      if (compact && (gemm_nt_ok(g) || !p.bf16)) {      // rows of padded frames: zero, and left out of the product
        fill_dx = !dx_cleared;
        g.a_rows = fidx; g.c_rows = fidx; g.a_phys_rows = TB; g.m_dev = count;
      }
      parts_dx = !p.bf16 || (gemm_tile_ok(g) && gemm_tile_small(g.M, g.N, g.nz));
    }
    // Weight gradients straight from the frame-major tensors (a row per frame in X, Hprev and DZ: both operands of
    // X^T DZ are k-major), over the packed list of real frames when lengths are given.
    auto frame_major = [&](const void* A, long lda, long sAz, int M, void* C) {
      GemmArgs g = {};
      g.A = A; g.B = DZ; g.C = C;
      g.M = M; g.N = 4 * p.n; g.K = (int)TB; g.lda = lda; g.ldb = 4 * n; g.ldc = 4 * n;
      g.sAz = sAz; g.sBz = (long)p.DZ_dir_elems; g.sCz = (long)M * 4 * n; g.nz = p.D; g.nseg = 1;
      g.a_kcontig = false; g.b_kcontig = false; g.in_bf16 = true; g.out_bf16 = false; g.accumulate = acc;
      if (compact) { g.k_rows = fidx; g.k_phys_rows = (int)TB; g.k_dev = count; }
      return g;
    };
    const bool pad_x = p.n_in8 != p.n_in;                          // rows of x are not 16-byte aligned: padded copy
    GemmArgs gx = frame_major(pad_x ? ws + p.ws_xpad : x, p.n_in8, 0, p.n_in, dW_x);
    GemmArgs gh = frame_major(rs + p.res_hprev, p.ldh, (long)(p.res_dir_stride / 2), p.n, dW_h);
    const auto frame_major_ok = [](const GemmArgs& g) { return gemm_tile_small(g.M, g.N, g.nz) ? gemm_tile_ok(g) : gemm_tn_ok(g); };
    const bool all_major = p.fast_gemm && (!seq_lens || compact) && frame_major_ok(gx) && frame_major_ok(gh);
    const auto in_few_tiles = [&]() {                              // both weight gradients; their parts' room is what is free now
      if (!all_major || !gemm_tile_small(gx.M, gx.N, gx.nz) || !gemm_tile_small(gh.M, gh.N, gh.nz)) return false;
      parts_of(gx);
      parts_of(gh);
      return gemm_tn_ranges(gx) == 1 && gemm_tn_ranges(gh) == 1;
    };
    const auto pad_x_rows = [&]() { return pad_x && !x_padded ? launch_pad_rows(x, ws + p.ws_xpad, (long)TB, p.n_in, p.n_in8, s) : hipSuccess; };
    if (dx) {
      const bool together = p.bf16 && parts_dx && in_few_tiles();
      Phase ph({{LSTM_PHASE_GEMM_DX, (double)p.n_in}, {LSTM_PHASE_GEMM_DWX, together ? (double)p.n_in : 0.0}, {LSTM_PHASE_GEMM_DWH, together ? (double)n : 0.0}}, 1, s);
      if (fill_dx) HIPCHK(launch_fill_zero(dx, (size_t)TB * n_in * p.esz, s));
      if (parts_dx) parts_of(gd);
      if (together) {
        HIPCHK(pad_x_rows());
        HIPCHK(launch_gemm_tile_grads(gd, gx, gh, s));
        return LSTM_OK;
      }
      HIPCHK(launch_gemm(gd, s));
    }
    if (all_major) {
      const bool pair = in_few_tiles();
      if (!pair && gemm_tile_small(gx.M, gx.N, gx.nz)) parts_of(gx);
      {
        Phase ph({{LSTM_PHASE_GEMM_DWX, (double)p.n_in}, {LSTM_PHASE_GEMM_DWH, pair ? (double)n : 0.0}}, 1, s);
        HIPCHK(pad_x_rows());
        if (pair) {
          HIPCHK(launch_gemm_tile_pair(gx, gh, s));
          return LSTM_OK;
        }
        HIPCHK(gemm_tn_ranges(gx) > 1 ? launch_gemm_tn_ranges(gx, s) : launch_gemm(gx, s));
      }
      Phase ph(LSTM_PHASE_GEMM_DWH, 1, s);
      if (gemm_tile_small(gh.M, gh.N, gh.nz)) parts_of(gh);
      HIPCHK(gemm_tn_ranges(gh) > 1 ? launch_gemm_tn_ranges(gh, s) : launch_gemm(gh, s));
    } else {                         // dW_x = X^T DZ, padded frames of X masked out
      GemmArgs g = {};
      g.A = x; g.B = DZ; g.C = dW_x;
      g.M = p.n_in; g.N = 4 * p.n; g.K = TB;
      g.lda = n_in; g.ldb = 4 * n; g.ldc = 4 * n;
      g.sAz = 0; g.sBz = (long)p.DZ_dir_elems; g.sCz = (long)(n_in * 4 * n); g.nz = p.D; g.nseg = 1;
      g.a_kcontig = false; g.b_kcontig = false; g.in_bf16 = p.bf16; g.out_bf16 = false; g.accumulate = acc;
      if (compact) { g.k_rows = fidx; g.k_phys_rows = (int)TB; g.k_dev = count; }   // the real frames only
      else { g.lens = seq_lens; g.Bt = p.B; g.T = p.T; }                              // (or every frame, padded ones read as zero)
      if (!p.bf16) {
        parts_of(g);
        if (pad_x) {
          GemmArgs gp = g;
          gp.A = ws + p.ws_xpad; gp.lda = p.n_in8;
          if (gemm_float_ok(gp)) {
            if (!x_padded) HIPCHK(launch_pad_rows(x, ws + p.ws_xpad, (long)TB, 2 * p.n_in, 2 * p.n_in8, s));
            g = gp;
          }
        }
      }
      {
        Phase ph(LSTM_PHASE_GEMM_DWX, 1, s);
        HIPCHK(launch_gemm(g, s));
      }
      // dW_h = Hprev^T DZ
      g.A = rs + p.res_hprev; g.C = dW_h; g.M = p.n; g.lda = p.ldh;
      g.sAz = (long)(p.res_dir_stride / p.esz); g.sCz = (long)(n * 4 * n);
      g.lens = nullptr;
      if (!p.bf16) parts_of(g);
      Phase ph(LSTM_PHASE_GEMM_DWH, 1, s);
      HIPCHK(launch_gemm(g, s));
    }
    return LSTM_OK;
  };
  if (p.dw_tiny) {
    Phase ph({{LSTM_PHASE_GEMM_DWX, (double)n_in}, {LSTM_PHASE_GEMM_DWH, (double)n}, {LSTM_PHASE_GEMM_DX, dx ? (double)n_in : 0.0}}, 1, s);
    HIPCHK(launch_gemm_tiny(tiny, p.bf16, (unsigned*)(ws + p.ws_tiny_cnt), (float*)(ws + p.ws_tiny_parts), s));
  } else if ((rc = products())) return rc;
  if (db_slices && !db_done) {
    SumJob j = {};
    j.parts = (const float*)(ws + p.ws_colsum); j.C = db; j.M = 1; j.N = 4 * p.n; j.ksplit = db_slices; j.nz = p.D;
    j.ldp = 4 * n; j.sPz = (long)kColsumSlices * 4 * n; j.ldc = 4 * n; j.sCz = 4 * n; j.accumulate = acc;
    sums.add(j);                         // (three products and this: the list holds four)
  }
  if (sums.count > 0) {                // one launch: its time by what each sum reads
    PhaseShare sh[4] = {{LSTM_PHASE_DB, 0}, {LSTM_PHASE_GEMM_DX, 0}, {LSTM_PHASE_GEMM_DWX, 0}, {LSTM_PHASE_GEMM_DWH, 0}};
    for (int i = 0; i < sums.count; ++i) {
      const SumJob& j = sums.j[i];
      sh[j.C == dx ? 1 : j.C == dW_x ? 2 : j.C == dW_h ? 3 : 0].weight += (double)j.M * j.N * j.nz * j.ksplit;
    }
    Phase ph({sh[0], sh[1], sh[2], sh[3]}, 1, s);
    HIPCHK(launch_sums(sums, s));
  }
  if (db_slices || db_done) return LSTM_OK;
  Phase ph(LSTM_PHASE_DB, 2, s);
  HIPCHK(launch_colsum(DZ, (float*)db, (float*)(ws + p.ws_colsum), TB, 4 * p.n, p.D, (long)p.DZ_dir_elems, p.bf16, acc, s));
  return LSTM_OK;
}

}  // namespace
int device_ok() { return check_device(); }
}  // namespace lstm

extern "C" {

int lstm_query(const lstm_desc* desc, int bidirectional, size_t* reserve_bytes, size_t* workspace_bytes) {
  lstm::Plan p;
  int rc = lstm::make_plan(desc, bidirectional, &p);
  if (rc) return rc;
  if (!reserve_bytes || !workspace_bytes) return LSTM_ERR_NULL;
  *reserve_bytes = (desc->flags & LSTM_FLAG_INFERENCE) ? 0 : p.reserve_bytes;
  *workspace_bytes = p.workspace_bytes;
  return LSTM_OK;
}

int lstm_fwd(const lstm_desc* desc, const void* x, const void* W_x, const void* W_h, const void* b, const void* h0,
             const void* c0, const int32_t* seq_lens, void* y, void* c, void* hT, void* cT, void* reserve, void* workspace,
             void* stream) {
  return lstm::run_fwd(desc, 0, x, W_x, W_h, b, h0, c0, seq_lens, y, c, hT, cT, reserve, workspace, stream);
}
int blstm_fwd(const lstm_desc* desc, const void* x, const void* W_x, const void* W_h, const void* b, const void* h0,
              const void* c0, const int32_t* seq_lens, void* y, void* c, void* hT, void* cT, void* reserve, void* workspace,
              void* stream) {
  return lstm::run_fwd(desc, 1, x, W_x, W_h, b, h0, c0, seq_lens, y, c, hT, cT, reserve, workspace, stream);
}
int lstm_bwd(const lstm_desc* desc, const void* x, const void* W_x, const void* W_h, const void* h0, const void* c0,
             const int32_t* seq_lens, const void* y, const void* c, const void* reserve, const void* dy, const void* dhT,
             const void* dcT, void* dx, void* dW_x, void* dW_h, void* db, void* dh0, void* dc0, void* workspace,
             void* stream) {
  return lstm::run_bwd(desc, 0, x, W_x, W_h, h0, c0, seq_lens, y, c, reserve, dy, dhT, dcT, dx, dW_x, dW_h, db, dh0, dc0,
                       workspace, stream);
}
int blstm_bwd(const lstm_desc* desc, const void* x, const void* W_x, const void* W_h, const void* h0, const void* c0,
              const int32_t* seq_lens, const void* y, const void* c, const void* reserve, const void* dy, const void* dhT,
              const void* dcT, void* dx, void* dW_x, void* dW_h, void* db, void* dh0, void* dc0, void* workspace,
              void* stream) {
  return lstm::run_bwd(desc, 1, x, W_x, W_h, h0, c0, seq_lens, y, c, reserve, dy, dhT, dcT, dx, dW_x, dW_h, db, dh0, dc0,
                       workspace, stream);
}

int lstm_gemm(int in_bf16, int out_bf16, int a_kcontig, int b_kcontig, int M, int N, int K, const void* A, int64_t lda,
              const void* B, int64_t ldb, void* C, int64_t ldc, const float* bias, int accumulate, const int32_t* lens,
              int Bt, int T, void* stream) {
  using namespace lstm;
  if (!A || !B || !C) return LSTM_ERR_NULL;
  if (M < 0 || N < 0 || K < 0 || lda < 1 || ldb < 1 || ldc < 1) return LSTM_ERR_DIM;
  if ((out_bf16 && !in_bf16) || (!a_kcontig && b_kcontig) || (lens && (a_kcontig || Bt < 1)) || (accumulate && out_bf16))
    return LSTM_ERR_UNSUPPORTED;
  const size_t esz = in_bf16 ? 2 : 4;
  if (((uintptr_t)A | (uintptr_t)B) & (esz - 1) || ((uintptr_t)C & (out_bf16 ? 1 : 3))) return LSTM_ERR_ALIGN;
  int rc = check_device();
  if (rc) return rc;
  GemmArgs g = {};
  g.A = A; g.B = B; g.C = C; g.bias = bias; g.M = M; g.N = N; g.K = K; g.lda = lda; g.ldb = ldb; g.ldc = ldc;
  g.nz = 1; g.nseg = 1; g.a_kcontig = a_kcontig; g.b_kcontig = b_kcontig; g.in_bf16 = in_bf16; g.out_bf16 = out_bf16;
  g.accumulate = accumulate; g.lens = lens; g.Bt = Bt; g.T = T;
  if (launch_gemm(g, (hipStream_t)stream) != hipSuccess) { (void)hipGetLastError(); return LSTM_ERR_HIP; }
  return LSTM_OK;
}

static int pool_args(int dtype, int T, int B, int F, int pool, const void* a, int64_t lda, const void* o, int64_t ldo) {
  if (!a || !o) return LSTM_ERR_NULL;
  if (T < 0 || B < 0 || F < 1 || pool < 1 || pool > 255 || lda < F || ldo < F || B > 65535) return LSTM_ERR_DIM;
  if (dtype != LSTM_F32 && dtype != LSTM_BF16_F32STATE) return LSTM_ERR_UNSUPPORTED;
  const uintptr_t mask = dtype == LSTM_F32 ? 3 : 1;
  if (((uintptr_t)a | (uintptr_t)o) & mask) return LSTM_ERR_ALIGN;
  return LSTM_OK;
}

int lstm_time_pool_fwd(int dtype, int T, int B, int F, int pool, const void* y, int64_t ldy, const int32_t* seq_lens, void* out,
                       int64_t ldo, uint8_t* arg, int32_t* lens_out, void* stream) {
  int rc = pool_args(dtype, T, B, F, pool, y, ldy, out, ldo);
  if (rc) return rc;
  if ((rc = lstm::check_device())) return rc;
  if (lstm::launch_time_pool_fwd(dtype == LSTM_BF16_F32STATE, y, ldy, seq_lens, out, ldo, arg, lens_out, T, B, F, pool,
                                 (hipStream_t)stream) != hipSuccess) {
    (void)hipGetLastError();
    return LSTM_ERR_HIP;
  }
  return LSTM_OK;
}

int lstm_time_pool_bwd(int dtype, int T, int B, int F, int pool, const void* dout, int64_t ldo, const uint8_t* arg,
                       const int32_t* seq_lens, void* dy, int64_t ldy, void* stream) {
  int rc = pool_args(dtype, T, B, F, pool, dout, ldo, dy, ldy);
  if (rc) return rc;
  if (!arg) return LSTM_ERR_NULL;
  if ((rc = lstm::check_device())) return rc;
  if (lstm::launch_time_pool_bwd(dtype == LSTM_BF16_F32STATE, dout, ldo, arg, seq_lens, dy, ldy, T, B, F, pool,
                                 (hipStream_t)stream) != hipSuccess) {
    (void)hipGetLastError();
    return LSTM_ERR_HIP;
  }
  return LSTM_OK;
}

int lstm_sync_status(const void* workspace, int32_t* timed_out) {
  if (!workspace || !timed_out) return LSTM_ERR_NULL;
  const char* ws = (const char*)(((uintptr_t)workspace + lstm::kAlign - 1) / lstm::kAlign * lstm::kAlign);
  uint32_t word = 0;
  if (hipMemcpy(&word, ws, 4, hipMemcpyDeviceToHost) != hipSuccess) { (void)hipGetLastError(); return LSTM_ERR_HIP; }
  *timed_out = word != 0;
  return LSTM_OK;
}

int lstm_profile_enable(int on) {
  lstm::g_profile = on < 0 ? 0 : on > 2 ? 2 : on;
  return LSTM_OK;
}
int lstm_profile_read(double* ms, int64_t* launches) {
  if (!ms || !launches) return LSTM_ERR_NULL;
  int rc = LSTM_OK;
  for (auto& r : lstm::g_recs) {
    float t = 0.f;
    if (hipEventSynchronize(r.e1) != hipSuccess || hipEventElapsedTime(&t, r.e0, r.e1) != hipSuccess) {
      (void)hipGetLastError();
      rc = LSTM_ERR_HIP;
    } else {
      double all = 0.0;
      for (int i = 0; i < r.count; ++i) all += r.share[i].weight;
      for (int i = 0; i < r.count; ++i) ms[r.share[i].phase] += t * (r.share[i].weight / all);
      launches[r.share[0].phase] += r.launches;
    }
    (void)hipEventDestroy(r.e0);
    (void)hipEventDestroy(r.e1);
  }
  lstm::g_recs.clear();
  return rc;
}

const char* lstm_strerror(int status) {
  switch (status) {
    case LSTM_OK: return "ok";
    case LSTM_ERR_NULL: return "a required pointer is NULL";
    case LSTM_ERR_DIM: return "bad dimension";
    case LSTM_ERR_DIRECTION: return "direction must be +1 or -1";
    case LSTM_ERR_UNSUPPORTED: return "unsupported dtype or flag";
    case LSTM_ERR_ALIGN: return "pointer is not 16-byte aligned";
    case LSTM_ERR_SIZE: return "reserve or workspace too small (see lstm_query)";
    case LSTM_ERR_HIP: return "HIP runtime error or device is not gfx950";
    default: return "unknown status";
  }
}

}  // extern "C"
