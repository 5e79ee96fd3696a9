// Host side of the cnn355 C ABI (include/cnn355.h): architecture grammar, shape inference
// (Sec. 2.2 Eq. 1), connection tables (Sec. 3.1), planning of the per-image step into stages,
// carving of the caller's workspace, and the entry points.  No device memory is allocated here.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cctype>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/cnn355.h"
#include "cnn355_dev.h"
#include "cnn355_flowspec.h"

namespace cnn355 {
hipError_t launch_stage(const Stage& st, const LayerDev& L, hipStream_t stream, const ProgramDev* d_prog, int s,
                        StatusDev* d_status, const RunArgs& a);
hipError_t launch_stage_pair(int kind_a, int n_a, int kind_b, int n_b, hipStream_t stream, const ProgramDev* d_prog,
                             int s, StatusDev* d_status, const RunArgs& a, bool* done);
hipError_t launch_reset_status(hipStream_t stream, StatusDev* d_status, int clear_label_flag);
hipError_t launch_call_set(hipStream_t stream, CallArgs* d_call, const CallArgs& v);
const void* call_advance_kernel();
const void* stage_kernel(const Stage& st, const LayerDev& L, int* threads);
int conv_bwd_win_group(int K, int KP);
const void* stage_pair_kernel(int kind_a, int kind_b);
hipError_t launch_persistent(int grid, bool with_matrix_stages, hipStream_t stream, const ProgramDev* d_prog,
                             StatusDev* d_status, const RunArgs& a);
int persistent_max_blocks_per_cu();
void read_dbg(unsigned long long* out);
hipError_t launch_frontend_batch(hipStream_t stream, const ProgramDev* d_prog, const float* d_images,
                                 long long image_stride, int n_images, int items_per_image, float* d_out);
hipError_t launch_crossing_probe(int G, int stride, hipStream_t stream, tagged_t* buf, int words, int rounds,
                                 unsigned int epoch_base, unsigned int spin_limit, StatusDev* d_status);
hipError_t launch_empty(hipStream_t stream, StatusDev* d_status);
hipError_t launch_resident(int static_id, int grid, size_t lds_bytes, hipStream_t stream, const FlowSpec& spec,
                           const FlowPtrs* d_ptrs, StatusDev* d_status, const RunArgs& a);
int resident_static_id(const FlowSpec& z);
size_t batch_gemm_lds_bytes(const BatchGemm& g);
hipError_t launch_batch_gemm(hipStream_t stream, const BatchGemm& g);
size_t batch_conv_lds_bytes(const BatchConv& g);
int batch_conv_fit(int MT, int TR, size_t lds_bytes);
int batch_conv_grid_x(const BatchConv& g);
hipError_t launch_batch_conv(hipStream_t stream, const BatchConv& g);
int batch_first_steps(int k_total);
size_t batch_first_lds_bytes(const BatchFirst& g);
int batch_first_fit(const BatchFirst& g);
hipError_t launch_batch_first(hipStream_t stream, const BatchFirst& g);
size_t batch_split_lds_bytes(const BatchSplit& g);
int batch_split_fit(const BatchSplit& g);
hipError_t launch_batch_split(hipStream_t stream, const BatchSplit& g);
hipError_t launch_batch_tail(hipStream_t stream, const BatchTail& g);
hipError_t launch_batch_pool(hipStream_t stream, const BatchPool& q);
hipError_t launch_batch_outputs(hipStream_t stream, const float* sums, int n_slices, long long slice_stride, const float* bias,
                                float* probs, long long n_images, int n_classes, int out_units);
hipError_t launch_batch_pack(hipStream_t stream, const BatchPackAll& all);
hipError_t launch_deform(hipStream_t stream, const DeformJob& J);
bool deform_mx_is_faster(const DeformJob& J);
}  // namespace cnn355

using namespace cnn355;

namespace {

constexpr int FE_BATCH = 256;  // images whose front-end outputs are computed ahead of the resident kernel

thread_local std::string g_err;  // message of the last failure that had no handle to carry it

struct ArchLayer {
  int kind = CNN_LAYER_INPUT;
  int maps = 0, h = 0, w = 0, K = 0, S = 0;  // K, S: the y (row) values of kernel / pooling rectangle and skipping factor
  int Kx = 0, Sx = 0;                        // their x (column) values
};

int fail(std::string* where, int code, const std::string& msg) {
  if (where) *where = msg;
  g_err = msg;
  return code;
}

// ---- grammar: <C>x<H>x<W> { -<M>C<K>[S<s>] | -MP<K> | -<N>N }+ ; K, s: <k> or <ky>x<kx> -------------
bool take_number(const std::string& s, size_t& pos, int& v) {
  if (pos >= s.size() || !std::isdigit((unsigned char)s[pos])) return false;
  long long x = 0;
  while (pos < s.size() && std::isdigit((unsigned char)s[pos])) {
    x = x * 10 + (s[pos] - '0');
    if (x > (1 << 20)) return false;
    ++pos;
  }
  v = (int)x;
  return true;
}

// <k> (both directions) or <ky>x<kx> (Sec. 2.2, 2.3: an x and a y value each)
bool take_pair(const std::string& s, size_t& pos, int& vy, int& vx) {
  if (!take_number(s, pos, vy)) return false;
  vx = vy;
  if (pos < s.size() && s[pos] == 'x') {
    ++pos;
    if (!take_number(s, pos, vx)) return false;
  }
  return true;
}

int parse_arch(const char* arch, std::vector<ArchLayer>& out, std::string* err) {
  if (!arch) return fail(err, CNN_E_ARG, "architecture string is NULL");
  const std::string s(arch);
  std::vector<std::string> tok;
  {
    size_t a = 0;
    while (true) {
      size_t b = s.find('-', a);
      tok.push_back(s.substr(a, b == std::string::npos ? std::string::npos : b - a));
      if (b == std::string::npos) break;
      a = b + 1;
    }
  }
  out.clear();
  {
    ArchLayer in;
    size_t p = 0;
    const std::string& t = tok[0];
    if (!take_number(t, p, in.maps) || p >= t.size() || t[p++] != 'x' || !take_number(t, p, in.h) ||
        p >= t.size() || t[p++] != 'x' || !take_number(t, p, in.w) || p != t.size())
      return fail(err, CNN_E_SYNTAX, "input must be <C>x<H>x<W>, got '" + t + "'");
    if (in.maps < 1 || in.h < 1 || in.w < 1) return fail(err, CNN_E_SHAPE, "empty input '" + t + "'");
    out.push_back(in);
  }
  bool fc_seen = false;
  for (size_t ti = 1; ti < tok.size(); ++ti) {
    const std::string& t = tok[ti];
    const ArchLayer prev = out.back();
    ArchLayer l;
    size_t p = 0;
    if (t.size() >= 2 && t[0] == 'M' && t[1] == 'P') {
      p = 2;
      if (!take_pair(t, p, l.K, l.Kx) || p != t.size()) return fail(err, CNN_E_SYNTAX, "bad pooling token '" + t + "'");
      if (prev.kind != CNN_LAYER_CONV)
        return fail(err, CNN_E_SYNTAX, "'" + t + "': max-pooling must follow a convolutional layer");
      if (l.K < 1 || l.Kx < 1) return fail(err, CNN_E_SHAPE, "'" + t + "': empty pooling rectangle");
      if (prev.h % l.K || prev.w % l.Kx)
        return fail(err, CNN_E_SHAPE, "'" + t + "': rectangle does not tile a " + std::to_string(prev.h) + "x" +
                                          std::to_string(prev.w) + " map");
      l.kind = CNN_LAYER_POOL;
      l.maps = prev.maps;
      l.h = prev.h / l.K;
      l.w = prev.w / l.Kx;
    } else {
      int n = 0;
      if (!take_number(t, p, n) || p >= t.size()) return fail(err, CNN_E_SYNTAX, "bad token '" + t + "'");
      const char c = t[p++];
      if (c == 'C') {
        if (!take_pair(t, p, l.K, l.Kx)) return fail(err, CNN_E_SYNTAX, "bad kernel size in '" + t + "'");
        if (p < t.size()) {
          if (t[p++] != 'S' || !take_pair(t, p, l.S, l.Sx) || p != t.size())
            return fail(err, CNN_E_SYNTAX, "bad skipping factor in '" + t + "'");
        }
        if (fc_seen) return fail(err, CNN_E_SYNTAX, "'" + t + "': convolution after a fully connected layer");
        if (n < 1 || l.K < 1 || l.Kx < 1) return fail(err, CNN_E_SHAPE, "'" + t + "': empty layer");
        l.kind = CNN_LAYER_CONV;
        l.maps = n;
        // Eq. 1 of Sec. 2.2, rounded down: the kernel stays completely inside the map
        l.h = prev.h >= l.K ? (prev.h - l.K) / (l.S + 1) + 1 : 0;
        l.w = prev.w >= l.Kx ? (prev.w - l.Kx) / (l.Sx + 1) + 1 : 0;
        if (l.h < 1 || l.w < 1)
          return fail(err, CNN_E_SHAPE, "'" + t + "': kernel larger than its " + std::to_string(prev.h) + "x" +
                                            std::to_string(prev.w) + " input");
      } else if (c == 'N') {
        if (p != t.size()) return fail(err, CNN_E_SYNTAX, "bad token '" + t + "'");
        if (n < 1) return fail(err, CNN_E_SHAPE, "'" + t + "': empty layer");
        l.kind = CNN_LAYER_FC;
        l.maps = n;
        l.h = l.w = 1;
        fc_seen = true;
      } else {
        return fail(err, CNN_E_SYNTAX, "bad token '" + t + "'");
      }
    }
    out.push_back(l);
  }
  if (out.size() < 2 || out.back().kind != CNN_LAYER_FC)
    return fail(err, CNN_E_SYNTAX, "the last layer must be fully connected (<N>N)");
  return CNN_OK;
}

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// Does a convolutional layer go to the matrix cores?  Only where the contraction is really dense:
// at least 64 output maps, at least 256 terms per output (input maps x kernel taps), and a map that
// one wavefront set can tile (32-pixel tiles, at most 4 per wavefront).  The table must be full.
bool mfma_shape_ok(int Mi, int K, int Mo, int Ho, int Wo) {
  const long long Kd = (long long)Mi * K * K, P = (long long)Ho * Wo;
  return Mo >= 64 && Kd >= 256 && P >= 16 && P <= MAX_TILE_PIX && (P + 31) / 32 <= (WG / 64) * 4;
}
// The same for the delta pull through such a layer, which is FP's mirror image when the skipping
// factor is 0: rows = input maps, contraction over (output map, tap), columns = input pixels.
bool mfma_bwd_shape_ok(int Mi, int K, int S, int Mo, int Hi, int Wi) {
  const long long Kd = (long long)Mo * K * K, P = (long long)Hi * Wi;
  return S == 0 && Mi >= 32 && Kd >= 256 && P >= 16 && P <= MAX_TILE_PIX && (P + 31) / 32 <= (WG / 64) * 4;
}
// Buffers in LDS of such a product (cnn355_dev.h) over pixels P, and the maps of a chunk of its slice of `per` maps: with two
// buffers half of the slice, so that the second half is fetched behind the first one's arithmetic, as far as they go (0: not
// even one).
int mfma_buffers(int mode, int P, int KK, int map) {
  return mode != CNN_MODE_PERSISTENT && P <= MFMA_ONE_TILE && mfma_chunk_fits(1, KK, map, 2) ? 2 : 1;
}
int mfma_chunk(int per, int KK, int map, int buffers) {
  // (a short slice in one: its arithmetic would not cover a second fetch.  63 nets, an image's step with every slice in halves 0.995 to
  // 1.05 of the time, with slices up to four times as long in one 0.99 to 1.03)
  int ic = buffers == 1 || (long long)per * (map + 32 * KK) <= 8192 ? per : (per + 1) / 2;
  while (ic > 0 && !mfma_chunk_fits(ic, KK, map, buffers)) --ic;
  return ic;
}
// Weight gradients of such a layer as a matrix product over the output pixels: rows = output maps,
// columns = (input map, tap); the deltas of 32 maps over the whole output map must fit in LDS next
// to at least one input map.
bool mfma_wgrad_shape_ok(int Mi, int K, int Mo, int Hi, int Wi, int Ho, int Wo) {
  const long long cols = (long long)Mi * K * K, P = (long long)Ho * Wo;
  // (measured: below some 300 000 weights the vector kernel, which visits the winners only, is as fast)
  return Mo >= 64 && cols >= 256 && Mo * cols >= 300000 && P >= 4 && 32 * (P + 2) + P + (long long)Hi * Wi + 64 <= LDS_FLOATS;
}
// A layer of many output maps on few input maps (the first layer): its product with activation and pooling in one stage
// (cnn355_first.h), from two tiles of 32 maps on (k_conv_fwd has an item per map there: 126 maps of 8 x 8 7.3 us, 5.4 so;
// 300 of 46 x 46 33.9, 9.4) and up to eight input maps (measured over 23 nets with 9 to 24: 0.85 to 1.20 of the vector kernels'
// whole step, mostly above).  A contraction of 256 and more is cut into slices instead.  LDS floats of a work item of 32 maps
// and `rows` conv rows.
long long conv_fwd_mx_floats(const LayerDev& L, int rows) {
  const int Kd = L.Mi * L.K * L.K, P = rows * L.Wo;
  return 32LL * ((Kd + 27) / 32 * 32 + 4) + ((Kd + 3) & ~3) + (long long)L.Mi * ((rows - 1) * (L.S + 1) + L.K) * L.Wi + 64LL * (P | 1);
}
bool conv_fwd_mx_ok(const LayerDev& L) {
  return !L.rect && L.full_table && L.Mo >= 64 && L.Mi <= 8 && L.Mi * L.K * L.K < 256 && conv_fwd_mx_floats(L, L.Kp) <= LDS_FLOATS;
}
// Conv rows of a work item's band: the fewest that leave one round of the compute units, as far as LDS goes; 0 where the vector
// kernel stays the better one.  That has all maps in one round up to a map per compute unit, while a wavefront of this one
// walks the whole contraction alone, and a lane a whole pooling window: with few items and many taps, or large windows on small
// maps, that is the longer way.  Measured over 280 nets, forward call, what the vector kernel takes longer: 83C6 on seven maps
// of 8 x 8 (9 items, 252 taps) -2.2 us, 69C5 on six of 18 x 18 (21 items, 150) -0.5, 87C5 on five of 22 x 22 (27, 125) +0.2, 211C7 on
// two of 51 x 51 (105, 98) +17; over 5 x 5 windows 191C3 with 20 x 20 pixels -1.5, 157C3 with 35 x 35 +5; over 7 x 7 ones 251C5 with 28 x 28
// -5.5, 129C7 with 42 x 42 +6.6; over 9 x 9 ones 203C6 with 18 x 18 -15, and with more maps than compute units 382C5 -3.
int conv_fwd_mx_rows(const LayerDev& L, int n_cu) {
  if (!conv_fwd_mx_ok(L)) return 0;
  const int RT = (L.Mo + 31) / 32;
  int rows = L.Kp;
  while (RT * ((L.Ho + rows - 1) / rows) > n_cu && rows + L.Kp <= L.Ho && conv_fwd_mx_floats(L, rows + L.Kp) <= LDS_FLOATS) rows += L.Kp;
  const int taps = L.Mi * L.K * L.K, items = RT * ((L.Ho + rows - 1) / rows), window = L.Kp * L.Kp;
  if (L.Mo <= n_cu ? taps > 6 * items || (window > 16 && L.Mo * L.Ho * L.Wo < 4200 * window) : L.Mo <= 2 * n_cu && window > 64) return 0;
  return rows;
}
// Its gradients: the whole input and the winners of JG output maps in LDS, at least a wavefront a map.  From two maps a work
// item on, when the vector kernel takes two rounds of the compute units (42 such nets 0.9 to 3.9 us a step faster, 71 with a map an item 3.4
// slower to 0.5 faster).
bool conv_wgrad_first_ok(const LayerDev& L, int JG) {
  const long long RP = L.Wi + ((L.K - L.Wi) % 32 + 32) % 32, MP = L.Hi * RP + ((L.K * L.K - L.Hi * RP) % 32 + 32) % 32;
  return conv_fwd_mx_ok(L) && JG >= 2 && JG <= WG / 64 && L.Mi * MP + 2LL * JG * L.Hp * L.Wp <= LDS_FLOATS;
}
// The same over the pooling winners, a lane per input map (cnn355_winners.h).  64 input maps lie in LDS pixel by pixel;
// below 32 input maps most lanes idle, below 9 winners a map the matrix product multiplies few zeros and stays (300C4 with
// its four winners: 11 us either way), without pooling there are none to skip (126 maps -> 208C4: 62.7 us an image with
// the dense product, 68.4 so).
bool win_wgrad_shape_ok(int Mi, int K, int Hi, int Wi, int Kp, int HW) {
  return Mi >= 32 && K >= 2 && K <= 5 && Kp >= 2 && HW >= 9 && (long long)Hi * Wi * 65 <= LDS_FLOATS;
}
// The delta pull over the winners (cnn355_winners.hip): kernels are compiled for these kernel sizes and pooling windows.
// Measured over 90 nets, an image's whole step against the matrix product: 64 and more input maps and 2^20 terms 0.70 to
// 1.0 of the time; fewer maps leave lanes idle (42 -> 235C4: 54.2 us, 57.1 so), five by five filters over 2 x 2 windows
// keep 240 registers and gain from 2^23 terms (93 -> 111C5: 57.5, 59.3; 94 -> 487C5: 112, 103), two by two ones have four
// terms a branch and win and lose by turns (282 -> 416C2 93 and 78, 381 -> 383C2 114 and 116).
bool win_bwd_shape_ok(int Mi, int K, int S, int Kp, int Mo, int HW) {
  const long long terms = (long long)Mi * Mo * HW * K * K;
  return S == 0 && Mi >= 64 && K >= 3 && K <= 5 && Kp >= 2 && Kp <= 4 && terms >= (K == 5 && Kp == 2 ? 1 << 23 : 1 << 20);
}
int ceil_log2(int v) {
  int l = 0;
  while ((1 << l) < v) ++l;
  return l;
}

// A bump allocator over the caller's workspace; with base == NULL it only measures.
struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base((char*)b) {}
  template <class T>
  T* take(size_t count) {
    off = align_up(off, 256);
    T* p = base ? (T*)(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

}  // namespace

struct BatchKept;

struct cnn {
  std::vector<ArchLayer> arch;
  std::vector<int> dev_of_arch;  // arch layer -> index in prog.layers (pool -> its conv), -1 for input
  std::vector<std::vector<uint8_t>> tables;  // per convolutional layer, [Mo][Mi]
  // fixed front-end
  int fe_n = 0, fe_K = 0, fe_src_n = 0;
  std::vector<float> fe_filters;
  std::vector<int> fe_src;

  ProgramDev prog;  // host copy with device pointers
  ProgramDev* d_prog = nullptr;
  StatusDev* d_status = nullptr;
  // stage mode: the launches of graph_images images as one graph, replayed (one for training, one forward only)
  CallArgs* d_call = nullptr;
  int graph_images = 0;         // 0: every stage of every image is launched by itself (the default: measured, a
                                //   replayed kernel node costs what a launch costs once the kernels do real work)
  hipGraphExec_t graph_exec[2] = {nullptr, nullptr};
  int graph_built_for[2] = {0, 0};
  float* d_weights = nullptr;
  float* d_grad = nullptr;
  float* d_fe_filters = nullptr;
  int* d_fe_src = nullptr;
  float* d_fe_out = nullptr;
  float* d_fe_batch = nullptr;  // resident mode: front-end outputs of FE_BATCH images at a time
  std::vector<std::shared_ptr<const BatchKept>> batch_kept;   // plans of the last batched forward calls, the last one first
  std::mutex batch_kept_lock;
  float* d_mm_part = nullptr;   // partial sums of the matrix-core forward pass (one layer at a time)
  size_t mm_part_floats = 0;
  int use_mfma = 1;
  int out_units = CNN_OUTPUT_SOFTMAX_XENT;
  struct ConvBuf {
    float *act, *out, *delta, *dact;
    uint8_t* arg;
    int *argyx, *csr_ptr, *csr_idx, *csc_ptr, *csc_j, *csc_slot;
  };
  struct FcBuf { float *act, *delta, *dact; };
  std::vector<ConvBuf> conv_buf;
  std::vector<FcBuf> fc_buf;
  struct HostTable { std::vector<int> csr_ptr, csr_idx, csc_ptr, csc_j, csc_slot; int max_conn = 0, max_back = 0; };
  std::vector<HostTable> host_tables;  // per convolutional layer, rebuilt by plan()

  // resident mode
  FlowSpec flow;                // the plan (plain integers); the resident kernel takes it by value
  FlowPtrs flow_ptrs;           // where the layers and the exchange buffers lie on the device
  FlowPtrs* d_flow_ptrs = nullptr;
  int flow_static_id = 0;       // > 0: the plan equals that of a kernel compiled for a fixed network
  // a resident kernel compiled for this handle's own network and loaded from a code object
  hipModule_t special_module = nullptr;
  hipFunction_t special_func = nullptr;
  FlowSpec special_plan;        // the plan that code object was compiled for
  bool special_active = false;  // the current plan equals it: calls go to special_func
  tagged_t* d_xbuf = nullptr;   // every exchange buffer, one after the other
  size_t xbuf_words = 0;
  bool flow_ok = false;
  std::string flow_why;         // why resident mode cannot run this network
  int team_ranks = 0, team_stride = 0;  // 0 = automatic
  unsigned long long epoch = 0; // images run in resident mode so far (their tags)

  size_t n_weights = 0, n_weights_max = 0;
  size_t image_size = 0;
  int n_classes = 0;
  hipStream_t stream = nullptr;
  int device = 0;               // the device that was current at cnn_create
  int mode = CNN_MODE_STAGES;
  int n_cu = 0, grid_override = 0, coop_ok = 0, max_blocks_per_cu = 1;
  unsigned int spin_limit = 1u << 22;
  int barrier_kind = 1;
  bool need_status_reset = true;
  std::string err;
};

namespace {

int hip_fail(cnn* net, hipError_t e, const char* what) {
  return fail(net ? &net->err : nullptr, CNN_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}
#define HIP_TRY(net, call)                                   \
  do {                                                       \
    hipError_t e_ = (call);                                  \
    if (e_ != hipSuccess) return hip_fail(net, e_, #call);   \
  } while (0)

// Lay the workspace out.  With net->d_* pointers filled when base != NULL.
size_t carve(cnn* net, void* base) {
  Carver c(base);
  const auto& A = net->arch;
  // upper bound on weights: every table full
  size_t nw = 0;
  for (size_t l = 1; l < A.size(); ++l) {
    if (A[l].kind == CNN_LAYER_CONV) nw += (size_t)A[l].maps * (1 + (size_t)A[l - 1].maps * A[l].K * A[l].Kx);
    if (A[l].kind == CNN_LAYER_FC) nw += (size_t)A[l].maps * (1 + (size_t)A[l - 1].maps * A[l - 1].h * A[l - 1].w);
  }
  net->n_weights_max = nw;
  net->d_prog = c.take<ProgramDev>(1);
  net->d_status = c.take<StatusDev>(1);
  net->d_call = c.take<CallArgs>(1);
  net->d_weights = c.take<float>(nw);
  net->d_grad = c.take<float>(nw);
  net->d_fe_filters = c.take<float>((size_t)A[0].maps * MAX_FRONTEND_K * MAX_FRONTEND_K);
  net->d_fe_src = c.take<int>(A[0].maps);
  net->d_fe_out = c.take<float>((size_t)A[0].maps * A[0].h * A[0].w);
  net->d_fe_batch = c.take<float>((size_t)FE_BATCH * A[0].maps * A[0].h * A[0].w);
  {
    size_t mm = 0;
    for (size_t l = 1; l < A.size(); ++l)
      if (A[l].kind == CNN_LAYER_CONV) {
        if (mfma_shape_ok(A[l - 1].maps, A[l].K, A[l].maps, A[l].h, A[l].w))
          mm = std::max(mm, (size_t)MFMA_MAX_SLICES * A[l].maps * A[l].h * A[l].w);
        if (l >= 2 && mfma_bwd_shape_ok(A[l - 1].maps, A[l].K, A[l].S, A[l].maps, A[l - 1].h, A[l - 1].w))
          mm = std::max(mm, (size_t)MFMA_MAX_SLICES * A[l - 1].maps * A[l - 1].h * A[l - 1].w);
      }
    net->d_mm_part = c.take<float>(mm);
    net->mm_part_floats = mm;
  }
  net->d_flow_ptrs = c.take<FlowPtrs>(1);
  {  // resident mode: tagged exchange buffers, sized for any team (see plan_flow for the split)
    size_t words = 0, last_maps = 0, first_fc = 0, n_fc_seen = 0;
    for (size_t l = 1; l < A.size(); ++l) {
      if (A[l].kind == CNN_LAYER_CONV) {
        const bool pooled = l + 1 < A.size() && A[l + 1].kind == CNN_LAYER_POOL;
        const size_t small = pooled ? (size_t)A[l + 1].maps * A[l + 1].h * A[l + 1].w : (size_t)A[l].maps * A[l].h * A[l].w;
        words += 3 * 2 * small;  // pooled outputs, deltas, winner coordinates; two images in flight
        words += 2 * 256 * (small / A[l].maps);  // pulled sums of the shares of a map's pull (fewer than 256 of them)
        words += 2 * (size_t)A[l].maps * A[l - 1].maps * (A[l].K * A[l].Kx + 4);  // adjusted filters on their way to the forward copies
        last_maps = A[l].maps;
      } else if (A[l].kind == CNN_LAYER_FC) {
        if (!first_fc) first_fc = A[l].maps;
        // a second fully connected layer held by columns: partial sums of up to 256 ranks, deltas of its inputs
        if (++n_fc_seen == 2) words += 2 * (size_t)256 * A[l].maps + 2 * (size_t)A[l - 1].maps * A[l - 1].h * A[l - 1].w;
      }
    }
    words += 2 * std::min<size_t>(last_maps, 256) * first_fc + 2 * first_fc;
    net->xbuf_words = words;
    net->d_xbuf = c.take<tagged_t>(words);
  }
  net->conv_buf.clear();
  net->fc_buf.clear();
  for (size_t l = 1; l < A.size(); ++l) {
    if (A[l].kind == CNN_LAYER_CONV) {
      // a pooling rectangle of one pixel is the identity: the pooled values are the activations
      const bool pooled = l + 1 < A.size() && A[l + 1].kind == CNN_LAYER_POOL && (A[l + 1].K > 1 || A[l + 1].Kx > 1);
      const size_t full = (size_t)A[l].maps * A[l].h * A[l].w;
      const size_t small = pooled ? (size_t)A[l + 1].maps * A[l + 1].h * A[l + 1].w : full;
      const size_t nc = (size_t)A[l].maps * A[l - 1].maps;
      cnn::ConvBuf b;
      b.act = c.take<float>(full);
      b.out = pooled ? c.take<float>(small) : b.act;
      b.delta = c.take<float>(small);
      b.dact = c.take<float>(small);
      b.arg = c.take<uint8_t>(small);
      b.argyx = c.take<int>(small);
      b.csr_ptr = c.take<int>(A[l].maps + 1);
      b.csr_idx = c.take<int>(nc);
      b.csc_ptr = c.take<int>(A[l - 1].maps + 1);
      b.csc_j = c.take<int>(nc);
      b.csc_slot = c.take<int>(nc);
      net->conv_buf.push_back(b);
    } else if (A[l].kind == CNN_LAYER_FC) {
      cnn::FcBuf b;
      b.act = c.take<float>(A[l].maps);
      b.delta = c.take<float>(A[l].maps);
      b.dact = c.take<float>(A[l].maps);
      net->fc_buf.push_back(b);
    }
  }
  return align_up(c.off, 256);
}

// Choose the band of conv rows one workgroup computes in the forward stage.
int plan_conv_fwd(const LayerDev& L, Stage& st, int n_cu, std::string* err) {
  const int Kp = L.Kp, Wo = L.Wo, Ho = L.Ho;
  const int target = 256;
  int rows = 0;
  if (Kp * Wo <= WG) {
    // the largest band of at most 256 pixels that still gives `want` work items; if no band does,
    // the smallest band (most items) of at least one wavefront of pixels
    const int want = 128;
    int max_rows = std::min(Ho, (WG / Wo) / Kp * Kp);
    for (int r = max_rows; r >= Kp; r -= Kp)
      if ((long long)L.Mo * ((Ho + r - 1) / r) >= want) { rows = r; break; }
    if (!rows) {
      rows = Kp;
      while (rows * Wo < 64 && rows + Kp <= max_rows) rows += Kp;
    }
    st.pix_per_thread = 1;
  } else {
    if (Kp * Wo > MAX_TILE_PIX) return fail(err, CNN_E_SHAPE, "convolutional map too wide for the forward kernel");
    rows = std::min(Ho, (MAX_TILE_PIX / Wo) / Kp * Kp);
    while (rows > Kp && (long long)L.Mo * ((Ho + rows - 1) / rows) < target) rows -= Kp;
    st.pix_per_thread = 2;
  }
  st.tile_rows = rows;
  st.n_tiles = (Ho + rows - 1) / rows;
  st.n_items = L.Mo * st.n_tiles;
  const int map_sz = ((rows - 1) * (L.S + 1) + L.K) * L.Wi;
  const int chunk = std::min({LDS_IN / map_sz, LDS_AUX / (L.K * L.Kx), L.max_conn});
  if (chunk < 1) return fail(err, CNN_E_SHAPE, "convolution input rows do not fit the LDS staging area");
  st.chunk = chunk;
  st.tw_log2 = ceil_log2(std::min(map_sz, WG));
  // A few items more than compute units would leave most units idle through a second round: then two (or
  // three) output maps per item, which share the staged input maps (full table, all of them in one chunk).
  st.rows_per_wg = 1;
  if (L.full_table && L.Mi <= chunk && st.n_items > n_cu && st.n_items <= 3 * n_cu && st.n_items % n_cu < n_cu / 2 && st.n_items % n_cu != 0) {
    const int mp = (st.n_items + n_cu - 1) / n_cu;
    st.rows_per_wg = mp;
    st.n_items = ((L.Mo + mp - 1) / mp) * st.n_tiles;
  }
  return CNN_OK;
}

// Forward (CSR), backward (CSC) and slot tables of one convolutional layer from its 0/1 table.
void build_tables(int Mo, int Mi, const std::vector<uint8_t>& table, cnn::HostTable& T) {
  T = cnn::HostTable();
  T.csr_ptr.assign(Mo + 1, 0);
  T.csc_ptr.assign(Mi + 1, 0);
  for (int j = 0; j < Mo; ++j) {
    for (int i = 0; i < Mi; ++i)
      if (table[(size_t)j * Mi + i]) T.csr_idx.push_back(i);
    T.csr_ptr[j + 1] = (int)T.csr_idx.size();
    T.max_conn = std::max(T.max_conn, T.csr_ptr[j + 1] - T.csr_ptr[j]);
  }
  for (int i : T.csr_idx) ++T.csc_ptr[i + 1];
  for (int i = 0; i < Mi; ++i) {
    T.max_back = std::max(T.max_back, T.csc_ptr[i + 1]);
    T.csc_ptr[i + 1] += T.csc_ptr[i];
  }
  T.csc_j.resize(T.csr_idx.size());
  T.csc_slot.resize(T.csr_idx.size());
  std::vector<int> at(T.csc_ptr.begin(), T.csc_ptr.end() - 1);
  for (int j = 0; j < Mo; ++j)
    for (int s = T.csr_ptr[j]; s < T.csr_ptr[j + 1]; ++s) {
      const int q = at[T.csr_idx[s]]++;
      T.csc_j[q] = j;
      T.csc_slot[q] = s;
    }
}

// Every size a kernel relies on, re-derived from the finished plan: a stage whose operands do
// not fit its LDS areas or its thread mapping is refused here, never launched.
int check_plan(cnn* net) {
  const ProgramDev& P = net->prog;
  auto bad = [&](int s, const char* what) {
    return fail(&net->err, CNN_E_SHAPE, "stage " + std::to_string(s) + ": " + what);
  };
  for (int s = 0; s < P.n_stages; ++s) {
    const Stage& st = P.stages[s];
    const LayerDev& L = P.layers[st.layer];
    if (st.n_items < 1) return bad(s, "no work items");
    switch (st.kind) {
      case ST_CONV_FWD: {
        const int P_max = st.tile_rows * L.Wo;
        const int map_sz = ((st.tile_rows - 1) * (L.S + 1) + L.K) * L.Wi;
        if (st.tile_rows < L.Kp || st.tile_rows % L.Kp) return bad(s, "row band not a multiple of the pooling size");
        if (st.pix_per_thread == 1 ? P_max > WG : P_max > MAX_TILE_PIX) return bad(s, "row band too large");
        if (st.pix_per_thread != 1 && st.pix_per_thread != 2) return bad(s, "bad pixels per thread");
        if (st.chunk < 1 || (long long)st.chunk * map_sz > LDS_IN) return bad(s, "input chunk exceeds the LDS input area");
        if (st.chunk * L.K * L.Kx > LDS_AUX) return bad(s, "filter chunk exceeds the LDS filter area");
        if (st.rows_per_wg < 1 || st.n_tiles * st.tile_rows < L.Ho || st.n_items != ((L.Mo + st.rows_per_wg - 1) / st.rows_per_wg) * st.n_tiles)
          return bad(s, "row bands do not cover the maps");
        if (st.rows_per_wg > 1 && (!L.full_table || L.Mi > st.chunk)) return bad(s, "output maps of one work item must share one chunk of input maps");
        if ((1 << st.tw_log2) > WG) return bad(s, "staging width");
        break;
      }
      case ST_CONV_BWD: {
        const int pt = 1 << st.tw_log2;
        if (st.chunk < 1 || (long long)st.chunk * (L.Ho + 1) * (L.Wo + 1) > LDS_IN) return bad(s, "delta chunk exceeds its LDS area");
        if (st.chunk * L.K * L.Kx > LDS_AUX) return bad(s, "filter chunk exceeds its LDS area");
        if (pt < 1 || pt > WG || st.n_tiles * pt < L.Hi * L.Wi || st.n_items != L.Mi * st.n_tiles) return bad(s, "pixel tiles do not cover the map");
        if (st.layer < 1) return bad(s, "no layer below");
        break;
      }
      case ST_CONV_WGRAD: {
        if (st.chunk < 1 || (long long)st.chunk * L.Hi * L.Wi > LDS_IN) return bad(s, "input maps exceed the LDS input area");
        if (L.Hp * L.Wp > LDS_AUX || L.Hp * L.Wp > LDS_AUX2) return bad(s, "pooled map exceeds its LDS area");
        if (st.n_tiles * st.chunk < L.max_conn || st.n_items != L.Mo * st.n_tiles) return bad(s, "chunks do not cover the connections");
        if ((1 << st.tw_log2) > WG) return bad(s, "staging width");
        break;
      }
      case ST_FC_FWD:
        if (st.rows_per_wg < 1 || st.rows_per_wg > WG / 64 || (st.rows_per_wg & (st.rows_per_wg - 1))) return bad(s, "rows per workgroup");
        if (st.n_items * st.rows_per_wg < L.n_out) return bad(s, "rows not covered");
        break;
      case ST_HEAD:
        if (L.n_out > LDS_AUX || L.n_out > LDS_AUX2 || st.n_items != 1) return bad(s, "output layer too wide");
        break;
      case ST_FC_BWD:
        if (L.n_out > LDS_AUX) return bad(s, "layer too wide");
        if (st.cm_log2 < 0 || st.cm_log2 > 8 || (st.n_items << st.cm_log2) < L.n_in) return bad(s, "columns not covered");
        break;
      case ST_FRONTEND:
        if (st.n_items * WG < P.fe.n_filters * P.fe.H * P.fe.W) return bad(s, "pixels not covered");
        break;
      case ST_CONV_FWD_MFMA: {
        const int KK = L.K * L.K, HiWi = L.Hi * L.Wi, Pn = L.Ho * L.Wo;
        const int NT = (Pn + 31) / 32, waves = WG / 64, KW = NT >= waves ? 1 : waves / NT;
        if (L.rect || !L.full_table || !mfma_shape_ok(L.Mi, L.K, L.Mo, L.Ho, L.Wo)) return bad(s, "layer not fit for the matrix-core kernel");
        if (st.tile_rows != mfma_buffers(net->mode, Pn, KK, HiWi) || !mfma_chunk_fits(st.chunk, KK, HiWi, st.tile_rows)) return bad(s, "chunk exceeds LDS");
        if (st.n_tiles < 1 || st.n_tiles > L.Mi || st.n_items != ((L.Mo + 31) / 32) * st.n_tiles) return bad(s, "slices do not cover the input maps");
        if (st.rows_per_wg != st.n_tiles || st.rows_per_wg > MFMA_MAX_SLICES) return bad(s, "too many partial-sum planes");
        if (KW > 1 && (long long)KW * NT * 1024 > LDS_FLOATS) return bad(s, "k splits do not fit LDS");
        if (((L.Mi + st.n_tiles - 1) / st.n_tiles) * (st.n_tiles - 1) >= L.Mi) return bad(s, "an empty slice");
        break;
      }
      case ST_CONV_BWD_MFMA: {
        const int KK = L.K * L.K, HWd = (L.Hi + L.K - 1) * (L.Wi + L.K - 1), Pn = L.Hi * L.Wi;
        const int NT = (Pn + 31) / 32, waves = WG / 64, KW = NT >= waves ? 1 : waves / NT;
        if (net->mode != CNN_MODE_STAGES) return bad(s, "the matrix-core pull is planned for the stage-launch mode only");
        if (L.rect || !L.full_table || !mfma_bwd_shape_ok(L.Mi, L.K, L.S, L.Mo, L.Hi, L.Wi)) return bad(s, "layer not fit for the matrix-core pull");
        if (st.tile_rows != mfma_buffers(net->mode, Pn, KK, HWd) || !mfma_chunk_fits(st.chunk, KK, HWd, st.tile_rows)) return bad(s, "chunk exceeds LDS");
        if (st.n_tiles < 1 || st.n_tiles > L.Mo || st.n_items != ((L.Mi + 31) / 32) * st.n_tiles) return bad(s, "slices do not cover the output maps");
        if (st.rows_per_wg != st.n_tiles || st.rows_per_wg > MFMA_MAX_SLICES) return bad(s, "too many partial-sum planes");
        if (KW > 1 && (long long)KW * NT * 1024 > LDS_FLOATS) return bad(s, "k splits do not fit LDS");
        if (((L.Mo + st.n_tiles - 1) / st.n_tiles) * (st.n_tiles - 1) >= L.Mo) return bad(s, "an empty slice");
        if (st.layer < 1 || P.layers[st.layer - 1].kind != L_CONV) return bad(s, "no convolutional layer below");
        break;
      }
      case ST_CONV_WGRAD_MFMA: {
        const int KK = L.K * L.K, Pn = L.Ho * L.Wo, WP = Pn + 1 + (Pn & 1);
        const int NT = (std::min(st.chunk, L.Mi) * KK + 31) / 32, waves = WG / 64, KW = NT >= waves ? 1 : waves / NT;
        if (net->mode != CNN_MODE_STAGES) return bad(s, "the matrix-core gradient is planned for the stage-launch mode only");
        if (L.rect || !L.full_table || !mfma_wgrad_shape_ok(L.Mi, L.K, L.Mo, L.Hi, L.Wi, L.Ho, L.Wo)) return bad(s, "layer not fit for the matrix-core gradient");
        if (st.chunk < 1 || (long long)st.chunk * L.Hi * L.Wi + 32LL * WP + Pn > LDS_FLOATS) return bad(s, "chunk exceeds LDS");
        if (NT > 4 * waves) return bad(s, "too many column tiles");
        if (KW > 1 && KW * NT * 1024 > LDS_FLOATS) return bad(s, "k splits do not fit LDS");
        if (st.n_tiles * st.chunk < L.Mi || (st.n_tiles - 1) * st.chunk >= L.Mi || st.n_items != ((L.Mo + 31) / 32) * st.n_tiles) return bad(s, "chunks do not cover the input maps");
        break;
      }
      case ST_CONV_WGRAD_WIN:
        if (net->mode != CNN_MODE_STAGES) return bad(s, "the gradient over the winners is planned for the stage-launch mode only");
        if (L.rect || !L.full_table || !win_wgrad_shape_ok(L.Mi, L.K, L.Hi, L.Wi, L.Kp, L.Hp * L.Wp)) return bad(s, "layer not fit for the gradient over the winners");
        if (st.chunk < 1 || st.chunk > WG / 64 || st.n_tiles * 64 < L.Mi || (st.n_tiles - 1) * 64 >= L.Mi || st.n_items != st.n_tiles * ((L.Mo + st.chunk - 1) / st.chunk))
          return bad(s, "work items do not cover the filters");
        break;
      case ST_CONV_FWD_MX:
        if (net->mode == CNN_MODE_PERSISTENT) return bad(s, "not in the persistent kernel");
        if (!conv_fwd_mx_ok(L) || st.tile_rows < L.Kp || st.tile_rows % L.Kp || conv_fwd_mx_floats(L, st.tile_rows) > LDS_FLOATS)
          return bad(s, "row band not fit for the matrix-core kernel");
        if (st.n_tiles * st.tile_rows < L.Ho || (st.n_tiles - 1) * st.tile_rows >= L.Ho || st.n_items != ((L.Mo + 31) / 32) * st.n_tiles)
          return bad(s, "row bands do not cover the maps");
        break;
      case ST_CONV_WGRAD_FIRST:
        if (net->mode != CNN_MODE_STAGES) return bad(s, "planned for the stage-launch mode only");
        if (!conv_wgrad_first_ok(L, st.chunk)) return bad(s, "layer not fit for the gradients of a first layer");
        if (st.n_items != (L.Mo + st.chunk - 1) / st.chunk) return bad(s, "work items do not cover the maps");
        break;
      case ST_CONV_BWD_WIN: {
        if (net->mode != CNN_MODE_STAGES) return bad(s, "the pull over the winners is planned for the stage-launch mode only");
        if (L.rect || !L.full_table || !win_bwd_shape_ok(L.Mi, L.K, L.S, L.Kp, L.Mo, L.Hp * L.Wp)) return bad(s, "layer not fit for the pull over the winners");
        const int NW = conv_bwd_win_group(L.K, L.Kp), NG = L.Hp * ((L.Wp + NW - 1) / NW);
        if (st.rows_per_wg < 1 || st.rows_per_wg > L.Mo || st.n_items != ((L.Mi + 63) / 64) * NG * st.rows_per_wg) return bad(s, "slices do not cover the output maps");
        if ((size_t)st.rows_per_wg * NG * (L.Kp + L.K - 1) * (L.Kp * NW + L.K - 1) * L.Mi > net->mm_part_floats) return bad(s, "partial sums exceed their scratch memory");
        if (st.layer < 1 || P.layers[st.layer - 1].kind != L_CONV) return bad(s, "no convolutional layer below");
        break;
      }
      case ST_CONV_BWD_WEPI:
        if (st.chunk < 1 || st.chunk > 64 || st.n_tiles != (L.Hi * L.Wi + st.chunk - 1) / st.chunk || st.n_items != ((L.Mi + 63) / 64) * st.n_tiles)
          return bad(s, "work items do not cover the input maps");
        if (s < 1 || P.stages[s - 1].kind != ST_CONV_BWD_WIN || st.rows_per_wg != P.stages[s - 1].rows_per_wg || st.tile_rows != conv_bwd_win_group(L.K, L.Kp))
          return bad(s, "not the sums of the stage before");
        break;
      case ST_CONV_BWD_EPI:
        if (st.rows_per_wg < 1 || st.rows_per_wg > MFMA_MAX_SLICES) return bad(s, "partial-sum planes");
        if (st.chunk < 1 || st.n_items != (L.Mi + st.chunk - 1) / st.chunk) return bad(s, "work items do not cover the input maps");
        if (st.layer < 1) return bad(s, "no layer below");
        break;
      case ST_CONV_EPI:
        if (st.rows_per_wg < 1 || st.rows_per_wg > MFMA_MAX_SLICES) return bad(s, "partial-sum planes");
        if (st.chunk < 1 || st.n_items != (L.Mo + st.chunk - 1) / st.chunk) return bad(s, "work items do not cover the maps");
        if (L.Ho * L.Wo > MAX_TILE_PIX) return bad(s, "map too large");
        if (st.chunk > 1 && st.chunk * L.Ho * L.Wo > WG) return bad(s, "maps of a work item exceed its lanes");
        break;
      default:
        return bad(s, "unknown stage kind");
    }
  }
  return CNN_OK;
}

void plan_flow(cnn* net);
void drop_stage_graphs(cnn* net);

// Build layer descriptors, tables and the stage list on the host (no device call).  Works on
// a handle whose workspace pointers are NULL (measuring / checking only).
int plan(cnn* net) {
  drop_stage_graphs(net);   // (their nodes carry the stage list that is about to change)
  const auto& A = net->arch;
  ProgramDev& P = net->prog;
  std::memset(&P, 0, sizeof(P));
  net->dev_of_arch.assign(A.size(), -1);
  net->host_tables.assign(net->tables.size(), cnn::HostTable());
  int nl = 0, conv_i = 0, fc_i = 0;
  std::vector<int> conv_of_dev(MAX_LAYERS, -1);  // descriptor index -> convolutional layer index
  size_t woff = 0;
  const float* below = nullptr;  // output buffer of the layer below
  const bool fe = net->fe_n > 0;
  bool has_below = fe;           // (pointers are all NULL when only measuring)
  if (fe) below = net->d_fe_out;
  for (size_t l = 1; l < A.size(); ++l) {
    if (A[l].kind == CNN_LAYER_POOL) { net->dev_of_arch[l] = nl - 1; continue; }
    if (nl >= MAX_LAYERS) return fail(&net->err, CNN_E_SHAPE, "too many layers");
    LayerDev& L = P.layers[nl];
    L.in_is_image = !has_below;
    L.in = below;
    if (A[l].kind == CNN_LAYER_CONV) {
      const bool pooled = l + 1 < A.size() && A[l + 1].kind == CNN_LAYER_POOL;
      L.kind = L_CONV;
      L.Mi = A[l - 1].maps; L.Hi = A[l - 1].h; L.Wi = A[l - 1].w;
      L.Mo = A[l].maps; L.Ho = A[l].h; L.Wo = A[l].w;
      L.K = A[l].K; L.S = A[l].S; L.Kx = A[l].Kx; L.Sx = A[l].Sx;
      L.Kp = pooled ? A[l + 1].K : 1;
      L.Kpx = pooled ? A[l + 1].Kx : 1;
      L.rect = (L.K != L.Kx || L.S != L.Sx || L.Kp != L.Kpx) ? 1 : 0;
      L.Hp = L.Ho / L.Kp; L.Wp = L.Wo / L.Kpx;
      if (L.Ho >= 65536 || L.Wo >= 65536) return fail(&net->err, CNN_E_SHAPE, "map too large");
      if (L.Hp * L.Wp > MAX_POOLED_PIX)
        return fail(&net->err, CNN_E_SHAPE, "pooled map has more than " + std::to_string(MAX_POOLED_PIX) + " positions");
      if (L.Hi * L.Wi > LDS_IN || (L.Ho + 1) * (L.Wo + 1) > LDS_IN)
        return fail(&net->err, CNN_E_SHAPE, "a map has more than " + std::to_string(LDS_IN) + " pixels");
      if (L.Kp > 15 || L.Kpx > 15) return fail(&net->err, CNN_E_SHAPE, "pooling rectangle larger than 15x15");
      const cnn::ConvBuf& b = net->conv_buf[conv_i];
      L.act = b.act; L.out = b.out; L.delta = b.delta; L.dact = b.dact; L.arg = b.arg; L.argyx = b.argyx;
      L.csr_ptr = b.csr_ptr; L.csr_idx = b.csr_idx; L.csc_ptr = b.csc_ptr; L.csc_j = b.csc_j; L.csc_slot = b.csc_slot;
      L.mm_part = net->d_mm_part;
      conv_of_dev[nl] = conv_i;
      build_tables(L.Mo, L.Mi, net->tables[conv_i], net->host_tables[conv_i]);
      L.max_conn = net->host_tables[conv_i].max_conn;
      L.full_table = net->host_tables[conv_i].csr_idx.size() == (size_t)L.Mo * L.Mi;
      const size_t n_conn = net->host_tables[conv_i].csr_idx.size();
      L.b_canon = (long long)woff;
      L.w_canon = (long long)(woff + L.Mo);
      woff += L.Mo + n_conn * L.K * L.Kx;
      ++conv_i;
    } else {
      L.kind = L_FC;
      L.n_in = A[l - 1].maps * A[l - 1].h * A[l - 1].w;
      L.n_out = A[l].maps;
      L.is_output = (l + 1 == A.size());
      L.out_units = L.is_output ? net->out_units : 0;
      if (L.n_out > MAX_FC_OUT)
        return fail(&net->err, CNN_E_SHAPE, "fully connected layer wider than " + std::to_string(MAX_FC_OUT));
      const cnn::FcBuf& b = net->fc_buf[fc_i];
      L.act = b.act; L.out = b.act; L.delta = b.delta; L.dact = b.dact;
      L.b_canon = (long long)woff;
      L.w_canon = (long long)(woff + L.n_out);
      woff += (size_t)L.n_out * (1 + (size_t)L.n_in);
      ++fc_i;
    }
    // (a handle that only plans, without a workspace, has no weights to point into)
    L.bias = net->d_weights ? net->d_weights + L.b_canon : nullptr;
    L.w = net->d_weights ? net->d_weights + L.w_canon : nullptr;
    below = L.out;
    has_below = true;
    net->dev_of_arch[l] = nl;
    ++nl;
  }
  P.n_layers = nl;
  P.n_classes = A.back().maps;
  net->n_classes = P.n_classes;
  net->n_weights = woff;
  P.has_frontend = fe ? 1 : 0;
  if (fe) {
    FrontendDev& F = P.fe;
    F.n_filters = net->fe_n; F.K = net->fe_K; F.n_src = net->fe_src_n;
    F.H = A[0].h; F.W = A[0].w;
    F.Hr = F.H + F.K - 1; F.Wr = F.W + F.K - 1;
    F.filters = net->d_fe_filters; F.src = net->d_fe_src; F.out = net->d_fe_out;
    net->image_size = (size_t)F.n_src * F.Hr * F.Wr;
  } else {
    net->image_size = (size_t)A[0].maps * A[0].h * A[0].w;
  }

  // ---- stage list ------------------------------------------------------------------------
  int ns = 0;
  auto add = [&](int kind, int layer, int n_items, int barrier, int train_only) -> Stage& {
    Stage& s = P.stages[ns++];
    s.kind = kind; s.layer = layer; s.n_items = n_items; s.barrier_after = barrier; s.train_only = train_only;
    return s;
  };
  if (4 * nl + 4 > MAX_STAGES) return fail(&net->err, CNN_E_SHAPE, "too many stages");
  if (fe) add(ST_FRONTEND, 0, (net->fe_n * A[0].h * A[0].w + WG - 1) / WG, 1, 0);
  for (int l = 0; l < nl; ++l) {  // forward, bottom up
    LayerDev& L = P.layers[l];
    const bool wide = L.kind == L_CONV && net->use_mfma && !L.rect && L.full_table && mfma_shape_ok(L.Mi, L.K, L.Mo, L.Ho, L.Wo);
    if (wide && L.Hi * L.Wi + 33 * L.K * L.K + 2 > LDS_FLOATS - 64)
      return fail(&net->err, CNN_E_SHAPE, "an input map does not fit the LDS staging area of the matrix-core kernel");
    // (a map or kernel of which half of LDS holds none, on few input maps: the product has nine work items at most, and the
    // vector kernel one for every output map and band of rows.  Measured, us an image forward, product and vector kernel:
    // 73C24S1 on one map of 46 x 102 (3 items) 59 and 38, 76C20S2 on three of 85 x 171 (9) 112 and 104, but 74C25S2 on four of
    // 31 x 164 (12) 43 and 45, 247C21S2 on three of 121 x 121 (24) 154 and 206)
    Stage by_band{};
    std::string why;
    const bool few = wide && !mfma_chunk_fits(1, L.K * L.K, L.Hi * L.Wi, 2) && (L.Mo + 31) / 32 * L.Mi <= 9 &&
                     plan_conv_fwd(L, by_band, net->n_cu > 0 ? net->n_cu : 256, &why) == CNN_OK;
    if (wide && !few) {
      // wide layer: implicit GEMM on the matrix cores, the contraction split over workgroups, then
      // a second stage that adds the partial sums and does what follows the sum
      const int n_cu = net->n_cu > 0 ? net->n_cu : 256;
      const int KK = L.K * L.K, HiWi = L.Hi * L.Wi, P = L.Ho * L.Wo;
      const int NT = (P + 31) / 32, waves = WG / 64;
      const int KW = NT >= waves ? 1 : waves / NT;
      const int RT = (L.Mo + 31) / 32;
      (void)KW;  // the k splits inside a workgroup are added there: one plane of partial sums per work item
      int KS = std::max(1, std::min({n_cu / RT, L.Mi, MFMA_MAX_SLICES}));
      const int per = (L.Mi + KS - 1) / KS;
      KS = (L.Mi + per - 1) / per;
      const int buffers = mfma_buffers(net->mode, P, KK, HiWi), IC = mfma_chunk(per, KK, HiWi, buffers);
      Stage& s = add(ST_CONV_FWD_MFMA, l, RT * KS, 1, 0);
      s.tile_rows = buffers;
      s.n_tiles = KS; s.chunk = IC; s.rows_per_wg = KS;
      // maps per work item of the second stage, side by side in its lanes: as many as leave every map its
      // lane groups (one per 8 planes, at most 4), and at least what brings the items down to one round of
      // the compute units where the lanes allow
      const int g_want = std::min((KS + 7) / 8, 4);
      const int mp_keep = std::max(1, WG / (P * g_want)), mp_need = (L.Mo + n_cu - 1) / n_cu;
      const int mp = P >= WG ? 1 : std::max(1, std::min({std::max(mp_keep, std::min(mp_need, WG / P)), L.Mo, 64}));
      Stage& e = add(ST_CONV_EPI, l, (L.Mo + mp - 1) / mp, 1, 0);
      e.rows_per_wg = KS;
      e.chunk = mp;
    } else if (int rows; L.kind == L_CONV && net->use_mfma && net->mode != CNN_MODE_PERSISTENT && (rows = conv_fwd_mx_rows(L, net->n_cu > 0 ? net->n_cu : 256)) > 0) {
      const int RT = (L.Mo + 31) / 32;
      Stage& s = add(ST_CONV_FWD_MX, l, 0, 1, 0);
      s.tile_rows = rows;
      s.n_tiles = (L.Ho + rows - 1) / rows;
      s.n_items = RT * s.n_tiles;
    } else if (L.kind == L_CONV) {
      Stage& s = add(ST_CONV_FWD, l, 0, 1, 0);
      int rc = plan_conv_fwd(L, s, net->n_cu > 0 ? net->n_cu : 256, &net->err);
      if (rc) return rc;
    } else if (!L.is_output) {
      Stage& s = add(ST_FC_FWD, l, 0, 1, 0);
      // lanes per neuron: about a quarter of its inputs (a few loads per lane), 64 .. 1024
      int lanes = 64;
      while (lanes < WG && lanes * 4 < L.n_in) lanes *= 2;
      s.rows_per_wg = WG / lanes;
      s.n_items = (L.n_out + s.rows_per_wg - 1) / s.rows_per_wg;
    } else {
      add(ST_HEAD, l, 1, 1, 0);
    }
  }
  // backward, top down.  The weights of a convolutional layer are adjusted one stage after the
  // deltas have been pulled through them; that adjustment shares a stage with the next pull.
  int pending_wgrad = -1;
  const bool matrix_stages = net->use_mfma && net->mode == CNN_MODE_STAGES;
  auto full = [&](const LayerDev& L) { return matrix_stages && !L.rect && L.full_table; };
  auto win_wgrad = [&](const LayerDev& L) { return full(L) && win_wgrad_shape_ok(L.Mi, L.K, L.Hi, L.Wi, L.Kp, L.Hp * L.Wp); };
  auto mfma_wgrad = [&](const LayerDev& L) { return full(L) && mfma_wgrad_shape_ok(L.Mi, L.K, L.Mo, L.Hi, L.Wi, L.Ho, L.Wo); };
  auto win_bwd = [&](const LayerDev& L) { return full(L) && win_bwd_shape_ok(L.Mi, L.K, L.S, L.Kp, L.Mo, L.Hp * L.Wp); };
  auto mfma_bwd = [&](const LayerDev& L) { return full(L) && mfma_bwd_shape_ok(L.Mi, L.K, L.S, L.Mo, L.Hi, L.Wi); };
  // (shared: the stage that follows is one that the adjustment has a launch with)
  auto add_wgrad = [&](int l, int barrier, bool shared) {
    LayerDev& L = P.layers[l];
    // compute units for one round of this stage's items next to those of the (short) stage launched with it
    const int n_cu_all = net->n_cu > 0 ? net->n_cu : 256;
    const bool after_epi = ns >= 1 && (P.stages[ns - 1].kind == ST_CONV_BWD_EPI || P.stages[ns - 1].kind == ST_CONV_BWD_WEPI);
    const int n_cu = after_epi ? std::max(n_cu_all / 2, n_cu_all - P.stages[ns - 1].n_items) : n_cu_all;
    // The winners' kernel has a work item for 64 input maps and an output map: where that is half a round of the compute units or
    // more, or the launch is another stage's as well.  Measured over 150 nets, an image's whole step against the kernels below:
    // 0.75 to 1.00 of the time from 128 items on; fewer that share a launch 0.90 to 1.03 (5 x 5 filters beside the sums of a pull
    // 0.98 to 1.06: not taken), with a launch of their own 1.00 to 1.03.
    const bool after_wgrad = ns >= 1 && !P.stages[ns - 1].barrier_after && (P.stages[ns - 1].kind == ST_CONV_WGRAD || P.stages[ns - 1].kind == ST_CONV_WGRAD_WIN);
    const bool win_pays = (L.Mi + 63) / 64 * L.Mo >= 128 || shared || after_wgrad || (after_epi && L.K <= 4);
    if (win_wgrad(L) && win_pays) {
      // one work item per compute unit: 64 input maps, as many output maps as that leaves
      Stage& s = add(ST_CONV_WGRAD_WIN, l, 0, barrier, 1);
      s.n_tiles = (L.Mi + 63) / 64;
      const int groups = std::max(1, std::min(L.Mo, n_cu / s.n_tiles));
      s.chunk = std::min(WG / 64, (L.Mo + groups - 1) / groups);   // (a wavefront each)
      s.n_items = s.n_tiles * ((L.Mo + s.chunk - 1) / s.chunk);
      return;
    }
    if (mfma_wgrad(L)) {
      // wide layer, one launch per stage: the gradients as a matrix product over the output pixels.
      // Input maps per work item: about one work item per compute unit, whole column tiles of 32
      // where the kernel size allows, at most 64 column tiles, and what LDS holds.
      const int KK = L.K * L.K, HiWi = L.Hi * L.Wi, Pn = L.Ho * L.Wo;
      const int RT = (L.Mo + 31) / 32;
      const int WP = Pn + 1 + (Pn & 1);
      const int ic_lds = (LDS_FLOATS - 64 - 32 * WP - Pn) / HiWi;
      int unit = 1;
      while ((unit * KK) % 32 != 0 && unit < 8) unit *= 2;   // a few maps that fill whole column tiles, if there are such
      if ((unit * KK) % 32 != 0) unit = 1;
      int ic = (L.Mi + std::max(1, n_cu / RT) - 1) / std::max(1, n_cu / RT);
      ic = (ic + unit - 1) / unit * unit;
      ic = std::max(1, std::min({ic, ic_lds, 64 * 32 / KK, L.Mi}));
      Stage& s = add(ST_CONV_WGRAD_MFMA, l, 0, barrier, 1);
      s.chunk = ic;
      s.n_tiles = (L.Mi + ic - 1) / ic;
      s.n_items = RT * s.n_tiles;
      return;
    }
    if (matrix_stages && conv_wgrad_first_ok(L, (L.Mo + n_cu - 1) / n_cu)) {
      Stage& s = add(ST_CONV_WGRAD_FIRST, l, 0, barrier, 1);
      s.chunk = (L.Mo + n_cu - 1) / n_cu;   // one round of the compute units
      s.n_items = (L.Mo + s.chunk - 1) / s.chunk;
      return;
    }
    Stage& s = add(ST_CONV_WGRAD, l, 0, barrier, 1);
    const int chunk_max = std::min(LDS_IN / (L.Hi * L.Wi), L.max_conn), KK = L.K * L.Kx, HW = L.Hp * L.Wp;
    // as many work items as fit one round on the compute units: the connection lists cut into
    // floor(CUs / maps) chunks
    auto chunk_for = [&](int cus) {
      const int want = std::max(1, cus / L.Mo);
      return std::max(1, std::min(chunk_max, (L.max_conn + want - 1) / want));
    };
    // (winners that a thread walks one by one)
    auto terms = [&](int chunk) {
      const int NW = chunk * KK, R = NW < WG ? std::max(1, std::min(WG / NW, HW)) : 1;
      return (HW + R - 1) / R * ((NW + WG - 1) / WG);
    };
    // next to the sums of a pull: shorter lists in more items, some of them behind the sums, where a thread's walk is that much
    // shorter (a term some 0.08 us, the sums 6: 48C8 on 36 maps, 512 winners for 1024, with the sums 44 us for 71; 13C5 on
    // 105 maps, 60 for 72, an image's step 139 us with the longer lists, 146 with the shorter)
    int chunk = chunk_for(n_cu);
    if (n_cu < n_cu_all && terms(chunk) > terms(chunk_for(n_cu_all)) + 75) chunk = chunk_for(n_cu_all);
    s.chunk = chunk;
    s.n_tiles = (L.max_conn + chunk - 1) / chunk;
    s.n_items = L.Mo * s.n_tiles;
    s.tw_log2 = ceil_log2(std::min(L.Hi * L.Wi, WG));
  };
  for (int l = nl - 2; l >= 0; --l) {  // layer nl-1 is the output layer, handled by ST_HEAD
    LayerDev& L = P.layers[l];
    if (L.kind == L_FC) {
      Stage& s = add(ST_FC_BWD, l, 0, 1, 1);
      // columns per work item: whole 256-byte (or 128-byte) pieces of a row of W where that still gives a third of the
      // compute units an item, else 64-byte pieces (5000 x 200 in pieces of 64, 128 and 256 bytes: 80.2, 78.7 and 78.5 us an
      // image, 3200 x 100 76.3 and 74.9)
      s.cm_log2 = (L.n_in / 64 >= 80) ? 6 : (L.n_in / 32 >= 80) ? 5 : 4;
      s.n_items = (L.n_in + (1 << s.cm_log2) - 1) >> s.cm_log2;
    } else {
      if (!L.in_is_image && l > 0) {
        // pull deltas into layer l-1 (reads the old weights of layer l) ...
        const bool with_pending = pending_wgrad >= 0;
        if (with_pending) { add_wgrad(pending_wgrad, 0, !win_bwd(L) && !mfma_bwd(L)); pending_wgrad = -1; }
        if (win_bwd(L)) {
          // wide layer, one launch per stage: the winners' terms only, a lane per input map; the contraction over the output maps
          // split so that there is about one work item per compute unit, as far as the scratch memory goes, 32 output maps or more each
          // (four to a wavefront; 33 nets, an image's step with 16 or more 0.97 to 1.02 of the time, with 64 or more 0.98 to 1.06)
          const int n_cu = net->n_cu > 0 ? net->n_cu : 256;
          const int NW = conv_bwd_win_group(L.K, L.Kp), NG = L.Hp * ((L.Wp + NW - 1) / NW), MC = (L.Mi + 63) / 64;
          const size_t region = (size_t)NG * (L.Kp + L.K - 1) * (L.Kp * NW + L.K - 1) * L.Mi;
          int KS = (int)std::min<size_t>(std::max(1, std::min(n_cu / (MC * NG), L.Mo / 32)), net->mm_part_floats / region);
          if (KS >= 1) {
            const int per = (L.Mo + KS - 1) / KS;
            KS = (L.Mo + per - 1) / per;
            Stage& s = add(ST_CONV_BWD_WIN, l, MC * NG * KS, 1, 1);
            s.rows_per_wg = KS;
            const int Pin = L.Hi * L.Wi;
            Stage& e = add(ST_CONV_BWD_WEPI, l, 0, 0, 1);
            e.rows_per_wg = KS;
            e.tile_rows = NW;
            // pixels of an item, for some 64 items beside the adjustment's: 16 at least (a wavefront each) and 64 at most (a lane each when
            // they are stored).  33 nets: at least 32 of them 0.98 to 1.06 of the step's time, some 128 items 0.97 to 1.07
            e.chunk = std::min(64, std::max(16, Pin * MC / 64));
            e.n_tiles = (Pin + e.chunk - 1) / e.chunk;
            e.n_items = MC * e.n_tiles;
            add_wgrad(l, 1, false);
            continue;
          }
        }
        if (mfma_bwd(L)) {
          // wide layer, one launch per stage (the persistent kernel does not hold this stage kind:
          // its registers would slow every other stage): the pull as FP's mirror image on the matrix cores, the contraction over the
          // output maps split over workgroups; the second stage adds the partial sums -- the
          // adjustment of this layer's weights, which the first stage has read, shares its interval
          const int n_cu = net->n_cu > 0 ? net->n_cu : 256;
          const int KK = L.K * L.K, HWd = (L.Hi + L.K - 1) * (L.Wi + L.K - 1);
          const int RT = (L.Mi + 31) / 32;
          int KS = std::max(1, std::min({n_cu / RT, L.Mo, MFMA_MAX_SLICES}));
          const int per = (L.Mo + KS - 1) / KS;
          KS = (L.Mo + per - 1) / per;
          const int buffers = mfma_buffers(net->mode, L.Hi * L.Wi, KK, HWd), IC = mfma_chunk(per, KK, HWd, buffers);
          if (IC >= 1) {
            Stage& s = add(ST_CONV_BWD_MFMA, l, RT * KS, 1, 1);
            s.tile_rows = buffers;
            s.n_tiles = KS; s.chunk = IC; s.rows_per_wg = KS;
            // input maps per work item of the second stage: up to two passes of the lanes over their pixels, but at
            // least 16 items (the weight adjustment that shares the interval leaves few compute units idle)
            const int Pin2 = L.Hi * L.Wi;
            const int mpb = std::max(1, std::min({2 * WG / Pin2, (L.Mi + 15) / 16, L.Mi}));
            Stage& e = add(ST_CONV_BWD_EPI, l, (L.Mi + mpb - 1) / mpb, 0, 1);
            e.rows_per_wg = KS;
            e.chunk = mpb;
            add_wgrad(l, 1, false);
            continue;
          }
        }
        Stage& s = add(ST_CONV_BWD, l, 0, 1, 1);
        const int Pin = L.Hi * L.Wi, HW = L.Hp * L.Wp, KK = L.K * L.Kx;
        const int max_back = net->host_tables[conv_of_dev[l]].max_back;
        // pixel tile: a power of two between 16 and 1024, small enough to give about 256 work items
        int pt = WG;
        while (pt > 16 && (pt / 2 >= Pin || (long long)L.Mi * ((Pin + pt - 1) / pt) < 256)) pt /= 2;
        s.tw_log2 = ceil_log2(pt);
        s.n_tiles = (Pin + pt - 1) / pt;
        s.n_items = L.Mi * s.n_tiles;
        s.chunk = std::max(1, std::min({LDS_IN / ((L.Ho + 1) * (L.Wo + 1)), LDS_AUX / KK, std::max(1, max_back)}));
        (void)HW;
        // ... then adjust the weights of layer l one stage later
        pending_wgrad = l;
      } else {
        // first trainable layer: nothing to pull; adjust it together with whatever is pending
        if (pending_wgrad >= 0) { add_wgrad(pending_wgrad, 0, win_wgrad(L) || !mfma_wgrad(L)); pending_wgrad = -1; }
        add_wgrad(l, 1, false);
      }
    }
  }
  if (pending_wgrad >= 0) { add_wgrad(pending_wgrad, 1, false); pending_wgrad = -1; }
  if (ns > 0) P.stages[ns - 1].barrier_after = 1;
  P.n_stages = ns;

  int rc = check_plan(net);
  if (rc) return rc;
  plan_flow(net);
  if (net->mode == CNN_MODE_RESIDENT && !net->flow_ok) {   // (its stages are other ones)
    net->mode = CNN_MODE_PERSISTENT;
    return plan(net);
  }
  return CNN_OK;
}


// Resident mode: choose the team, lay out every rank's LDS (flow_plan, shared with the kernels that
// are compiled for fixed networks) and the exchange buffers.  Sets net->flow_ok; a network the mode
// cannot take keeps flow_ok = false with the reason in flow_why (not an error: the other modes
// still run it).
void plan_flow(cnn* net) {
  const ProgramDev& P = net->prog;
  FlowSpec& Z = net->flow;
  FlowPtrs& Q = net->flow_ptrs;
  std::memset(&Z, 0, sizeof(Z));
  std::memset(&Q, 0, sizeof(Q));
  net->flow_ok = false;
  net->flow_static_id = 0;
  net->special_active = false;
  auto no = [&](const std::string& why) { net->flow_why = why; };
  int n_conv = 0;
  while (n_conv < P.n_layers && P.layers[n_conv].kind == L_CONV) ++n_conv;
  const int n_fc = P.n_layers - n_conv;
  if (n_conv < 1) return no("resident mode needs at least one convolutional layer");
  if (n_conv > FLOW_MAX_CONV || n_fc > FLOW_MAX_FC || n_fc < 1)
    return no("resident mode takes at most " + std::to_string(FLOW_MAX_CONV) + " convolutional and " +
              std::to_string(FLOW_MAX_FC) + " fully connected layers");
  Z.n_conv = n_conv; Z.n_fc = n_fc; Z.n_classes = P.n_classes; Z.out_units = net->out_units;
  for (int l = 0; l < n_conv; ++l) {
    const LayerDev& L = P.layers[l];
    if (L.rect) return no("resident mode takes kernels, skipping factors and pooling rectangles with equal x and y values only");
    ConvSpec& C = Z.conv[l];
    C.Mi = L.Mi; C.Hi = L.Hi; C.Wi = L.Wi; C.Mo = L.Mo; C.Ho = L.Ho; C.Wo = L.Wo;
    C.K = L.K; C.S = L.S; C.Kp = L.Kp; C.Hp = L.Hp; C.Wp = L.Wp;
    C.max_conn = L.max_conn; C.max_back = net->host_tables[l].max_back; C.full_table = L.full_table;
  }
  for (int f = 0; f < n_fc; ++f) {
    const LayerDev& L = P.layers[n_conv + f];
    Z.fc[f].n_in = L.n_in; Z.fc[f].n_out = L.n_out; Z.fc[f].is_output = L.is_output;
  }
  switch (flow_plan(Z, net->team_ranks, net->team_stride, net->n_cu)) {
    case FLOW_OK: break;
    case FLOW_BAD_STRIDE: return no("team stride must be 1 or 8");
    case FLOW_TOO_LARGE: return no("a layer is too large for resident mode");
    case FLOW_NO_LDS: return no("the weights and maps one workgroup would hold exceed its LDS");
    default: return no("resident mode cannot run this network");
  }
  // pointers: layers, tables, exchange buffers
  tagged_t* xb = net->d_xbuf;
  size_t xoff = 0;
  auto xtake = [&](size_t words) { tagged_t* p = xb ? xb + xoff : nullptr; xoff += words; return p; };
  for (int l = 0; l < n_conv; ++l) {
    const LayerDev& L = P.layers[l];
    FlowConvPtrs& C = Q.conv[l];
    C.w = L.w; C.bias = L.bias; C.act = L.act; C.out = L.out; C.arg = L.arg; C.argyx = L.argyx; C.delta = L.delta;
    C.csr_ptr = L.csr_ptr; C.csr_idx = L.csr_idx; C.csc_ptr = L.csc_ptr; C.csc_j = L.csc_j; C.csc_slot = L.csc_slot;
    C.w_canon = L.w_canon; C.b_canon = L.b_canon;
    const size_t small = (size_t)L.Mo * L.Hp * L.Wp;
    C.x_out = (l + 1 < n_conv) ? xtake(2 * small) : nullptr;
    C.x_delta = (l >= 1) ? xtake(2 * small) : nullptr;
    C.x_yx = (l >= 1) ? xtake(2 * small) : nullptr;
    C.x_part = (l >= 1 && Z.conv[l].pull_shares > 1)
                   ? xtake((size_t)2 * L.Mi * (Z.conv[l].pull_shares - 1) * L.Hi * L.Wi) : nullptr;
    C.x_w = (l >= 1 && Z.stream) ? xtake((size_t)2 * net->host_tables[l].csr_idx.size() * (L.K * L.K + 4)) : nullptr;
  }
  for (int f = 0; f < n_fc; ++f) {
    const LayerDev& L = P.layers[n_conv + f];
    FlowFcPtrs& C = Q.fc[f];
    C.w = L.w; C.bias = L.bias; C.act = L.act; C.delta = L.delta; C.w_canon = L.w_canon; C.b_canon = L.b_canon;
    C.x_part = nullptr; C.x_dprev = nullptr;
    if (Z.fc[f].by_cols) {
      C.x_part = xtake((size_t)2 * std::min(Z.G, Z.fc[f].n_in) * Z.fc[f].n_out);
      C.x_dprev = xtake((size_t)2 * Z.fc[f].n_in);
    }
  }
  Q.xp = xtake((size_t)2 * Z.n_col_ranks * Z.fc[0].n_out);
  Q.xsum = xtake((size_t)2 * Z.fc[0].n_out);
  if (xoff > net->xbuf_words) return no("internal: exchange buffers exceed their workspace area");
  if (xb && !Q.xp) return no("internal: an exchange buffer was not laid out");
  net->flow_static_id = resident_static_id(Z);
  net->special_active = net->special_func != nullptr && std::memcmp(&Z, &net->special_plan, sizeof(FlowSpec)) == 0;
  net->flow_ok = true;
  net->flow_why.clear();
}

// Upload what plan() built.  Weights are zeroed.
int upload(cnn* net) {
  const ProgramDev& P = net->prog;
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  int conv_i = 0;
  for (int l = 0; l < P.n_layers; ++l) {
    const LayerDev& L = P.layers[l];
    if (L.kind != L_CONV) continue;
    const cnn::HostTable& T = net->host_tables[conv_i];
    const cnn::ConvBuf& b = net->conv_buf[conv_i];
    HIP_TRY(net, hipMemcpy(b.csr_ptr, T.csr_ptr.data(), T.csr_ptr.size() * 4, hipMemcpyHostToDevice));
    HIP_TRY(net, hipMemcpy(b.csr_idx, T.csr_idx.data(), T.csr_idx.size() * 4, hipMemcpyHostToDevice));
    HIP_TRY(net, hipMemcpy(b.csc_ptr, T.csc_ptr.data(), T.csc_ptr.size() * 4, hipMemcpyHostToDevice));
    HIP_TRY(net, hipMemcpy(b.csc_j, T.csc_j.data(), T.csc_j.size() * 4, hipMemcpyHostToDevice));
    HIP_TRY(net, hipMemcpy(b.csc_slot, T.csc_slot.data(), T.csc_slot.size() * 4, hipMemcpyHostToDevice));
    if (L.Kp == 1 && L.Kpx == 1) {  // no pooling: every neuron is its own winner
      std::vector<int> yx((size_t)L.Mo * L.Ho * L.Wo);
      for (int j = 0; j < L.Mo; ++j)
        for (int y = 0; y < L.Ho; ++y)
          for (int x = 0; x < L.Wo; ++x) yx[((size_t)j * L.Ho + y) * L.Wo + x] = (y << 16) | x;
      HIP_TRY(net, hipMemcpy(L.argyx, yx.data(), yx.size() * 4, hipMemcpyHostToDevice));
      HIP_TRY(net, hipMemset(L.arg, 0, yx.size()));
    }
    ++conv_i;
  }
  HIP_TRY(net, hipMemcpy(net->d_prog, &P, sizeof(P), hipMemcpyHostToDevice));
  HIP_TRY(net, hipMemcpy(net->d_flow_ptrs, &net->flow_ptrs, sizeof(FlowPtrs), hipMemcpyHostToDevice));
  HIP_TRY(net, hipMemset(net->d_xbuf, 0, net->xbuf_words * sizeof(tagged_t)));
  net->epoch = 0;
  HIP_TRY(net, hipMemset(net->d_weights, 0, net->n_weights_max * sizeof(float)));
  HIP_TRY(net, hipMemset(net->d_status, 0, sizeof(StatusDev)));
  return CNN_OK;
}

int rebuild(cnn* net) {
  int rc = plan(net);
  if (rc) return rc;
  return upload(net);
}

// Plan for another mode and hand the stage list to the device where it is another one (else nothing is waited for, as long
// as no graph of launches is kept); weights, tables and everything else there stay.  A plan that fails leaves the handle as it was.
int replan(cnn* net, int mode) {
  const int old_mode = net->mode;
  const ProgramDev before = net->prog;
  net->mode = mode;
  const int rc = plan(net);
  if (rc) {
    const std::string why = net->err;
    net->mode = old_mode;
    (void)plan(net);
    net->err = why;
    return rc;
  }
  if (std::memcmp(&before, &net->prog, sizeof before) == 0) return CNN_OK;
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  HIP_TRY(net, hipMemcpy(net->d_prog, &net->prog, sizeof(ProgramDev), hipMemcpyHostToDevice));
  HIP_TRY(net, hipMemcpy(net->d_flow_ptrs, &net->flow_ptrs, sizeof(FlowPtrs), hipMemcpyHostToDevice));
  return CNN_OK;
}

int check_status(cnn* net) {
  StatusDev s;
  HIP_TRY(net, hipMemcpy(&s, net->d_status, sizeof(s), hipMemcpyDeviceToHost));
  int rc = CNN_OK;
  if (s.abort_flag) rc = fail(&net->err, CNN_E_HIP, "a wait inside the persistent or resident kernel timed out; the weights are undefined");
  else if (s.bad_label) rc = fail(&net->err, CNN_E_ARG, "a label outside [0, classes) was met; that image was skipped");
  if (s.abort_flag || s.bad_label) {
    const float loss = s.loss;
    std::memset(&s, 0, sizeof(s));
    s.loss = loss;
    HIP_TRY(net, hipMemcpy(net->d_status, &s, sizeof(s), hipMemcpyHostToDevice));
  }
  return rc;
}

int sync_and_check(cnn* net) {
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  return check_status(net);
}

int persistent_grid(const cnn* net, int train) {
  if (net->grid_override > 0) return std::min(net->grid_override, net->n_cu * net->max_blocks_per_cu);
  int most = 1;
  for (int s = 0; s < net->prog.n_stages; ++s)
    if (train || !net->prog.stages[s].train_only) most = std::max(most, net->prog.stages[s].n_items);
  return std::max(1, std::min(most, net->n_cu));
}

void drop_stage_graphs(cnn* net) {
  if (net->graph_exec[0] || net->graph_exec[1]) (void)hipStreamSynchronize(net->stream);  // (replays may be in flight)
  for (int w = 0; w < 2; ++w) {
    if (net->graph_exec[w]) (void)hipGraphExecDestroy(net->graph_exec[w]);
    net->graph_exec[w] = nullptr;
    net->graph_built_for[w] = 0;
  }
}

// The stage launches of `images` consecutive images as a chain of kernel nodes behind one node that moves the
// call's image counter on; every stage node carries its image's place in the graph, the rest comes from *d_call.
int build_stage_graph(cnn* net, int which, int images, const RunArgs& a0) {
  const ProgramDev& P = net->prog;
  if (net->graph_exec[which]) { (void)hipGraphExecDestroy(net->graph_exec[which]); net->graph_exec[which] = nullptr; }
  hipGraph_t graph = nullptr;
  HIP_TRY(net, hipGraphCreate(&graph, 0));
  auto give_up = [&](hipError_t e, const char* what) { (void)hipGraphDestroy(graph); return hip_fail(net, e, what); };
  hipGraphNode_t prev = nullptr;
  auto add = [&](const void* fn, unsigned grid, unsigned block, void** params) -> hipError_t {
    hipKernelNodeParams kp;
    std::memset(&kp, 0, sizeof(kp));
    kp.func = const_cast<void*>(fn);
    kp.gridDim = dim3(grid); kp.blockDim = dim3(block); kp.sharedMemBytes = 0; kp.kernelParams = params; kp.extra = nullptr;
    hipGraphNode_t node = nullptr;
    hipError_t e = hipGraphAddKernelNode(&node, graph, prev ? &prev : nullptr, prev ? 1 : 0, &kp);
    prev = node;
    return e;
  };
  {
    CallArgs* d_call = net->d_call;
    int step = images;
    void* params[] = {(void*)&d_call, (void*)&step};
    hipError_t e = add(call_advance_kernel(), 1, 64, params);
    if (e != hipSuccess) return give_up(e, "graph node (image counter)");
  }
  const ProgramDev* d_prog = net->d_prog;
  StatusDev* d_status = net->d_status;
  for (int i = 0; i < images; ++i) {
    RunArgs b = a0;
    b.call = net->d_call; b.t_local = i;
    b.images = nullptr; b.labels = nullptr; b.probs_out = nullptr; b.grad_out = nullptr; b.n_images = 1;
    for (int s = 0; s < P.n_stages; ++s) {
      const Stage& st = P.stages[s];
      if (st.train_only && !which) continue;
      if (st.n_items <= 0) continue;
      int stage = s;
      void* params[] = {(void*)&d_prog, (void*)&stage, (void*)&d_status, (void*)&b};
      if (!st.barrier_after && s + 1 < P.n_stages && P.stages[s + 1].train_only == st.train_only && P.stages[s + 1].n_items > 0) {
        const Stage& nx = P.stages[s + 1];
        if (const void* fn = stage_pair_kernel(st.kind, nx.kind)) {
          hipError_t e = add(fn, (unsigned)(st.n_items + nx.n_items), WG, params);
          if (e != hipSuccess) return give_up(e, "graph node (pair of stages)");
          ++s;
          continue;
        }
      }
      int threads = 0;
      const void* fn = stage_kernel(st, P.layers[st.layer], &threads);
      if (!fn) return give_up(hipErrorInvalidValue, "graph node (unknown stage)");
      hipError_t e = add(fn, (unsigned)st.n_items, (unsigned)threads, params);
      if (e != hipSuccess) return give_up(e, "graph node (stage)");
    }
  }
  hipGraphExec_t exec = nullptr;
  hipError_t e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
  (void)hipGraphDestroy(graph);
  if (e != hipSuccess) return hip_fail(net, e, "hipGraphInstantiate");
  net->graph_exec[which] = exec;
  net->graph_built_for[which] = images;
  return CNN_OK;
}

// The resident kernel of this handle: the one loaded for its own network when the plan is still the one that was
// compiled for, else a compiled-in one (for a benchmark network, or the one that reads its plan).
static hipError_t launch_resident_of(cnn* net, int grid, size_t lds_bytes, const RunArgs& a) {
  if (!net->special_active)
    return launch_resident(net->flow_static_id, grid, lds_bytes, net->stream, net->flow, net->d_flow_ptrs, net->d_status, a);
  RunArgs args = a;
  FlowSpec plan = net->flow;
  const FlowPtrs* d_ptrs = net->d_flow_ptrs;
  StatusDev* d_status = net->d_status;
  void* params[] = {(void*)&plan, (void*)&d_ptrs, (void*)&d_status, (void*)&args};
  return hipModuleLaunchCooperativeKernel(net->special_func, (unsigned)grid, 1, 1, WG, 1, 1, (unsigned)lds_bytes, net->stream, params);
}

// Does a forward call of so few images take the launches of its stages in resident mode too?  A cooperative launch costs some
// 25 us beside its kernel's work, and the kernel loads a rank's weights first; a stage costs some 6 us an image.  Measured, us
// (resident, stages): one image of the digits net 35, 24, two 44, 48; with the kernel that reads its plan, two of
// 100 maps a layer (7 launches) 90, 80, three 116, 121; three of 30 to 50 maps (5 launches) 103, 92.
bool forward_by_stages(const cnn* net, unsigned long long n) {
  int launches = 0;
  for (int s = 0; s < net->prog.n_stages; ++s) launches += net->prog.stages[s].train_only ? 0 : 1;
  const bool literal = net->flow_static_id > 0 || net->special_active;
  return n <= (literal ? 1u : launches > 5 ? 2u : 3u);
}

int run(cnn* net, const RunArgs& a0) {
  RunArgs a = a0;
  a.spin_limit = net->spin_limit;
  a.barrier_kind = net->barrier_kind;
  const ProgramDev& P = net->prog;
  if (net->mode == CNN_MODE_RESIDENT && (a.train || !forward_by_stages(net, (unsigned long long)a.n_images))) {
    const unsigned long long n = (unsigned long long)a.n_images;
    if (n >= (1ull << 31)) return fail(&net->err, CNN_E_ARG, "too many images in one call");
    if (((net->epoch + n) >> 32) != (net->epoch >> 32)) {
      // the 32-bit tags would wrap inside this call: start a fresh range on cleared buffers
      net->epoch = ((net->epoch >> 32) + 1) << 32;
      HIP_TRY(net, hipStreamSynchronize(net->stream));
      HIP_TRY(net, hipMemset(net->d_xbuf, 0, net->xbuf_words * sizeof(tagged_t)));
    }
    const int grid = net->flow.G * net->flow.stride;
    const size_t lds_bytes = (size_t)net->flow.lds_floats * sizeof(float);
    // (no launch clears the abort flag first: it is clear unless a call before this one gave up, whose error the next
    // synchronising call returns; until then the weights are undefined and the calls in between leave early)
    if (!P.has_frontend) {
      a.epoch_base = (unsigned int)net->epoch;
      net->epoch += n;
      HIP_TRY(net, launch_resident_of(net, grid, lds_bytes, a));
      return CNN_OK;
    }
    // fixed front-end: computed for FE_BATCH images at a time by all compute units, outside the
    // on-line chain; the resident kernel then trains on its outputs
    const size_t fe_sz = (size_t)P.fe.n_filters * P.fe.H * P.fe.W;
    const int items = (int)((fe_sz + WG - 1) / WG);
    for (unsigned long long t0 = 0; t0 < n; t0 += FE_BATCH) {
      const int nb = (int)std::min<unsigned long long>(FE_BATCH, n - t0);
      HIP_TRY(net, launch_frontend_batch(net->stream, net->d_prog, a0.images + t0 * a0.image_stride, a0.image_stride,
                                         nb, items, net->d_fe_batch));
      RunArgs b = a;
      b.images = net->d_fe_batch;
      b.image_stride = (long long)fe_sz;
      b.labels = a.labels ? a.labels + t0 : nullptr;
      b.probs_out = a.probs_out ? a.probs_out + t0 * P.n_classes : nullptr;
      b.n_images = nb;
      b.epoch_base = (unsigned int)net->epoch;
      net->epoch += (unsigned long long)nb;
      HIP_TRY(net, launch_resident_of(net, grid, lds_bytes, b));
      if (t0 + nb >= n)  // parity tap: layer 0 of the last image
        HIP_TRY(net, hipMemcpyAsync(net->d_fe_out, net->d_fe_batch + (size_t)(nb - 1) * fe_sz, fe_sz * sizeof(float),
                                    hipMemcpyDeviceToDevice, net->stream));
    }
    return CNN_OK;
  }
  if (net->mode == CNN_MODE_PERSISTENT) {
    bool mm = false;
    for (int s = 0; s < P.n_stages; ++s) {
      const int kind = P.stages[s].kind;
      const bool matrix = kind == ST_CONV_FWD_MFMA || kind == ST_CONV_EPI;
      // (the kernel would pass over a stage it does not hold)
      if (kind > ST_CONV_WGRAD && !matrix) return fail(&net->err, CNN_E_STATE, "internal: stage " + std::to_string(s) + " is not in the persistent kernel");
      mm = mm || matrix;
    }
    HIP_TRY(net, launch_reset_status(net->stream, net->d_status, 0));
    HIP_TRY(net, launch_persistent(persistent_grid(net, a.train), mm, net->stream, net->d_prog, net->d_status, a));
    return CNN_OK;
  }
  const long long n = a.n_images;
  long long t_first = 0;
  const int GB = net->graph_images;
  if (GB > 0 && a.labels && !a.grad_out && n >= 2 * GB) {
    // whole graphs of GB images first; what is left over is launched stage by stage below
    const int which = a.train ? 1 : 0;
    if (!net->graph_exec[which] || net->graph_built_for[which] != GB) {
      int rc = build_stage_graph(net, which, GB, a);
      if (rc) return rc;
    }
    CallArgs c;
    c.images = a.images; c.labels = a.labels; c.probs_out = a.probs_out; c.image_stride = a.image_stride;
    c.t0 = -(long long)GB; c.lr = a.lr; c.train = a.train;
    HIP_TRY(net, launch_call_set(net->stream, net->d_call, c));
    const long long n_graphs = n / GB;
    for (long long g = 0; g < n_graphs; ++g) HIP_TRY(net, hipGraphLaunch(net->graph_exec[which], net->stream));
    t_first = n_graphs * GB;
  }
  for (long long t = t_first; t < n; ++t) {
    RunArgs b = a;
    b.images = a.images + t * a.image_stride;
    b.labels = a.labels ? a.labels + t : nullptr;
    b.probs_out = a.probs_out ? a.probs_out + t * P.n_classes : nullptr;
    b.n_images = 1;
    for (int s = 0; s < P.n_stages; ++s) {
      const Stage& st = P.stages[s];
      if (st.train_only && !a.train) continue;
      if (!st.barrier_after && s + 1 < P.n_stages && P.stages[s + 1].train_only == st.train_only) {
        // the next stage does not depend on this one: both in one launch, where a kernel for the pair exists
        const Stage& nx = P.stages[s + 1];
        bool done = false;
        HIP_TRY(net, launch_stage_pair(st.kind, st.n_items, nx.kind, nx.n_items, net->stream, net->d_prog, s,
                                       net->d_status, b, &done));
        if (done) { ++s; continue; }
      }
      HIP_TRY(net, launch_stage(st, P.layers[st.layer], net->stream, net->d_prog, s, net->d_status, b));
    }
  }
  return CNN_OK;
}

}  // namespace

// ---- batched forward pass ------------------------------------------------------------------
namespace {

struct BatchStep {
  BatchGemm g;
  BatchConv c;        // used instead of g when c.MT != 0
  BatchFirst f;       // used instead of both when f.T != 0 ...
  BatchSplit s;       // ... or s.RT != 0
  BatchPool pool;     // used when the sums come raw (g.fuse or c.fuse 0)
  BatchPack pack;
  size_t wt_off = 0;  // floats from the start of the scratch
  size_t wt_floats = 0;
  size_t out_per_image = 0;   // floats an image in the layer's buffer
  bool split_out = false;     // outputs as split halves, for the next layer's product, and their marks behind them
  size_t halves_per_image = 0;   // floats an image of the halves
  bool raw() const { return s.RT ? s.raw : f.T == 0 && (c.MT ? c.fuse : g.fuse) == 0; }
};
struct BatchPlan {
  std::vector<BatchStep> steps;
  bool tail = false;   // the last two layers are k_batch_tail's (the first of them up to its sums)
  size_t wt_total = 0, sums_per_image = 0, act_per_image[2] = {0, 0}, fe_per_image = 0;   // (layers take the two buffers in turn)
  size_t floats(size_t batch) const {
    return wt_total + batch * (sums_per_image + act_per_image[0] + act_per_image[1] + fe_per_image) + 4 * 64;
  }
  size_t asked = 0;    // floats that a caller is asked for
};

size_t up64(size_t x) { return (x + 63) / 64 * 64; }

// Whether the output units add the planes of their own layer's sums: a launch less, but a thread adds all of an image's,
// class after class, eight planes at a time.  us with / without: 5 classes of 5 planes 45.4 / 46.1, of 19 49.3 / 48.4; 10 of
// 5 50.5 / 49.6, of 63 123 / 95 (a batch of 512); 2 of 38 27.0 / 27.6.
bool outputs_add(int n_classes, int n_planes) { return n_classes * ((n_planes + 7) / 8) <= 8; }

FastDiv fast_div_of(int d) {
  FastDiv f = {0, 0};
  while ((1ll << f.s) < d) ++f.s;
  f.m = (unsigned)(((1ull << (31 + f.s)) + (unsigned)d - 1) / (unsigned)d);
  return f;
}

// Time models of the two kernels for a convolutional layer, in clocks of a compute unit: coefficients fitted to the
// difference of the two kernels over 12700 layers, random ones and those of the benchmark's nets (1 to 300 maps of 1 to 96
// pixels, kernels 1 to 7, pooling to 12, batches to 10000).  k_batch_conv is the slower one by more than 3 % in 683 of
// them, in 143 of those that conv_plan gives it, which does without 0.4 % of what the kernel gains over all of them.  The
// more workgroups work side by side on a compute unit (1, 2, up to 4, more), the more of a workgroup's waits is hidden.
int side_by_side(double workgroups, int fit) {
  const double n = std::min((double)fit, workgroups);
  return n < 2 ? 0 : n < 3 ? 1 : n < 5 ? 2 : 3;
}
// k_batch_gemm: per chunk the products (k padded to whole groups) and the rounds of eight loads a thread that stage it
double gemm_clocks(const BatchGemm& g, size_t batch) {
  constexpr double ROUND[4] = {810, 850, 530, 90};
  const int rows = g.MT * g.TR, kc = g.IC * g.K * g.Kx, kg = g.TR == 32 ? 8 : 16, members = g.Kp * g.Kpx;
  const int regs = g.MT * (g.TR == 32 ? 16 : 8) * (members > 1 ? 2 : 1) + 80;
  const int fit = std::max(1, std::min({512 / regs, (int)(160 * 1024 / batch_gemm_lds_bytes(g)), 8}));
  const double side = std::ceil(std::ceil((double)batch * g.P / 128) * (g.MoPad / rows) * g.KS / 256);
  const int s = side_by_side(side, fit);
  const double images = std::min<double>((double)batch, 1.0 + 127.0 / g.P);
  const double rounds = std::ceil(images * g.IC * g.Hi * g.Wi / 2048) + std::ceil((kc + 1.0) * rows / 4096);
  const double chunk = 1600.0 + 0.82 * ((kc + kg - 1) / kg * kg) * rows * members + (g.prefetch ? 310.0 : ROUND[s]) * rounds;
  return side * (g.chunks_per_slice * chunk + 81.0 * rows) * (s ? 1.0 : 1.5) + (g.fuse == 0 ? 6400.0 : 0.0);
}
// k_batch_conv: per chunk the products and a wavefront's staging loads (a run of every image the block touches); per block
// a constant and the stores of its rows, or the tiles that pass through LDS.  A workgroup takes its blocks one after the
// other, the workgroups of a compute unit share its matrix cores.
double conv_clocks(const BatchConv& t, size_t batch, size_t n_cb) {
  constexpr double LOAD16[4] = {139, 126, 104, 104}, LOAD4[4] = {87, 78, 62, 66}, BLOCK[4] = {1930, 1290, 1220, 970};
  const int rows = t.MT * t.TR, kc = t.IC * t.K * t.Kx, kg = t.TR == 32 ? 8 : 16, HiWi = t.Hi * t.Wi, M = t.Kp * t.Kpx;
  const int fit = batch_conv_fit(t.MT, t.TR, batch_conv_lds_bytes(t));
  const size_t lines = (size_t)((t.Mo + rows - 1) / rows) * t.n_slices, gx = std::min(n_cb, std::max<size_t>(1, 256 * fit / lines));
  const size_t side = (gx * lines + 255) / 256, rounds = (n_cb + gx - 1) / gx;
  const int s = side_by_side((double)side, fit);
  const bool vec = (t.IC * HiWi) % 4 == 0 && t.in_stride % 4 == 0 && (t.n_slices == 1 || (t.run * HiWi) % 4 == 0);
  const double images = std::min<double>((double)batch, 1.0 + (t.wins - 1.0) / t.win_img);
  const int runs = (t.IC * HiWi + (vec ? 255 : 63)) / (vec ? 256 : 64);
  const double chunk = 0.78 * ((kc + kg - 1) / kg * kg) * rows + (vec ? LOAD16 : LOAD4)[s] * images * ((runs + 3) / 4);
  const double block = (t.run + t.IC - 1) / t.IC * chunk + BLOCK[s] + (M == 1 ? 49.0 * rows : M == 4 ? 0.0 : 285.0 * t.MT);
  return (double)(side * rounds) * block * (s ? 1.0 : 1.5) + (t.fuse == 0 ? 9700.0 : 0.0);
}

// The plan of k_batch_conv for a convolutional layer whose k_batch_gemm plan is g: the tile and chunk of the fewest clocks.
// Never more scratch memory than g takes: no more padded maps.  The slices of the k range are g's own, so that a running
// sum is no longer than there (fewer slices are faster for 33 stereo pairs, 77 us instead of 88, but the error of 128 maps
// of 450 terms in one sum instead of three is 3.6e-7 instead of 2.3e-7, that of 100 maps of 2500 terms in one instead of
// five 8.3e-7 instead of 4.1e-7; and ten and ten input maps instead of sixteen and four already 2.9e-7 instead of 2.8e-7).
// Leaves c.MT = 0 where a chunk of one input map does not fit, and where the models have k_batch_gemm as fast (or a tenth
// slower; sliced sums, where they err most, 5 % faster): this kernel stages image by image, so that blocks of many small
// images (layers of one output pixel) or of a small part of a large one leave its matrix cores waiting (5000 images, 100C4
// on 100 maps of 4 x 4: k_batch_gemm 118 us, k_batch_conv 223; 1289 of 1x81x81-4C6-MP2 433 and 704).
void conv_plan(const LayerDev& L, const BatchGemm& g, size_t batch, BatchConv& c) {
  constexpr size_t LDS_HALF = 80 * 1024, LDS_WHOLE = 158 * 1024;   // two workgroups a compute unit, or one
  std::memset(&c, 0, sizeof(c));
  BatchConv t;
  std::memset(&t, 0, sizeof(t));
  t.Mi = L.Mi; t.Hi = L.Hi; t.Wi = L.Wi; t.K = L.K; t.Kx = L.Kx; t.stride = L.S + 1; t.stride_x = L.Sx + 1; t.Mo = L.Mo;
  t.in_stride = g.in_stride; t.bias = L.bias; t.k_total = L.Mi * L.K * L.Kx;
  const int HiWi = L.Hi * L.Wi, members = L.Kp * L.Kpx;
  const size_t limit = (size_t)1 << 31;
  if ((size_t)HiWi * 4 * L.Mi >= limit || (size_t)t.k_total * 160 * 4 >= limit) return;   // (32-bit offsets of a chunk)
  double best = 0;
  const int slices = g.KS;
  t.n_slices = slices; t.run = std::min(t.Mi, g.chunks_per_slice * g.IC);
  // pooling inside, unless the k range is sliced or whole windows leave more than a quarter of the 128 columns empty
  const bool inside = slices == 1 && (members == 1 || (members <= 128 && 128 / members * members >= 96));
  if (!inside && members > 1 && g.fuse != 0) return;           // (g has no room for raw sums)
  t.Kp = inside ? L.Kp : 1; t.Kpx = inside ? L.Kpx : 1;
  t.Wp = inside ? L.Wp : L.Wo;
  t.win_img = inside ? L.Hp * L.Wp : L.Ho * L.Wo;
  t.wins = inside ? 128 / members : 128;
  t.fuse = slices > 1 || (!inside && members > 1) ? 0 : (L.is_output ? 2 : 1);
  const size_t n_cb = (batch * t.win_img + t.wins - 1) / t.wins;
  t.n_img_max = (int)std::min<size_t>(std::max<size_t>(batch, 1), (size_t)((t.wins - 1 + t.win_img - 1) / t.win_img + 1));
  for (int tr : {32, 16})
    for (int mt = tr == 32 ? 5 : 7; mt >= 1; --mt) {
      const int rows = mt * tr, groups = (t.Mo + rows - 1) / rows;
      if (groups * rows > g.MoPad) continue;
      t.TR = tr; t.MT = mt;
      for (size_t budget : {LDS_HALF, LDS_WHOLE}) {
        bool any = false;
        for (int ic = 1; ic <= t.run; ++ic) {   // (the last chunk of a slice may be short)
          t.IC = ic; t.slot = (int)up64((size_t)ic * HiWi); t.resident = ic == t.run;
          if (batch_conv_lds_bytes(t) > budget) {
            if (ic == t.run) break;
            ic = t.run - 1;      // the longest chunk may fit again: it needs its weights once
            continue;
          }
          any = true;
          const double est = conv_clocks(t, batch, n_cb);
          if (best == 0 || est < best) { best = est; c = t; }
        }
        if (any) break;
      }
    }
  if (best >= (c.fuse ? 1.1 : 0.95) * gemm_clocks(g, batch)) c.MT = 0;
  if (c.MT) { c.by_win_img = fast_div_of(c.win_img); c.by_wp = fast_div_of(c.Wp); }
}

// k_batch_split's clocks of a compute unit for a layer, fitted to 12 layers in up to 110 plans each: its workgroups share the
// matrix pipes and LDS, and each waits for its own slabs.  The plan of the fewest clocks takes 0 to 6 % longer (of the pass
// around the layer) than the fastest one.
double split_clocks(const BatchSplit& t, size_t n_cb) {
  const int S = t.TR == 32 ? 2 : 4, rows = t.RT * t.TR, cols = 4 * t.CT * t.TR, chunks = t.cps, slices = (t.n_cg / t.IC + t.cps - 1) / t.cps;
  const double steps = (double)chunks * (t.n_kg / S), slabs = (double)chunks * ((t.n_kg + t.slab - 1) / t.slab);
  const double matrix = steps * t.RT * t.CT * 3 * (t.TR == 32 ? 32 : 16), lds = steps * S * (rows + cols / 4);
  const size_t groups = (size_t)((t.Mo + rows - 1) / rows) * slices, gx = std::min(n_cb, std::max<size_t>(1, 256 * batch_split_fit(t) / groups));
  const double side = (double)((gx * groups + 255) / 256), rounds = (double)((n_cb + gx - 1) / gx);
  return rounds * std::max(side * (1.28 * matrix + 0.55 * lds + 263.0 * slabs + 60.0), 1.8 * matrix + 17.5 * steps + 1010.0 * slabs + 1330.0);
}

// The plan of k_batch_split for a convolutional layer behind another one: the tile, chunk and slab of the fewest clocks.  Leaves
// t.RT = 0 where windows do not fit a block, or leave more than a quarter of it empty, and where one group of eight maps of a
// block's images does not fit.
double split_plan(const LayerDev& L, size_t batch, BatchSplit& out) {
  constexpr size_t LDS = 160 * 1024;
  BatchSplit t;
  std::memset(&t, 0, sizeof(t));
  out = t;
  t.n_cg = (L.Mi + 7) / 8; t.pix = L.Hi * L.Wi; t.Wi = L.Wi; t.K = L.K; t.Kx = L.Kx; t.stride = L.S + 1; t.stride_x = L.Sx + 1;
  t.Mo = L.Mo; t.Kp = L.Kp; t.Kpx = L.Kpx; t.Wp = L.Wp; t.win_img = L.Hp * L.Wp; t.bias = L.bias;
  const int M = t.Kp * t.Kpx, KK = t.K * t.Kx;
  const size_t limit = (size_t)1 << 29, in_floats = (size_t)t.n_cg * 8 * t.pix;
  if (L.is_output || batch * in_floats >= limit || batch * (size_t)((L.Mo + 7) / 8 * 8) * t.win_img >= limit) return 0;
  t.in_plane = (long long)batch * t.pix * 16;   // (layers of halves stay below 2^31 bytes: the kernels' offsets)
  double best = 0;
  // pixels from a block's first to its last, at most, by the row of windows that it starts in
  int span_of = 0, span = 0;
  auto pixels = [&](int wins) {
    if (wins == span_of) return span;
    span_of = wins; span = 0;
    const int more_rows = wins % t.Wp == 0 ? wins / t.Wp - 1 : (wins + t.Wp - 2) / t.Wp;   // (blocks of whole rows start with one)
    for (int y = 0; y < L.Hp; ++y) {
      const int last = y + more_rows, rows = last / L.Hp * L.Hi + (last % L.Hp * t.Kp + t.Kp - 1) * t.stride + t.K - y * t.Kp * t.stride;
      span = std::max(span, rows * t.Wi);
    }
    return span = (int)std::min<size_t>((size_t)span, batch * t.pix);
  };
  for (int tr : {32, 16})
    for (int rt : {1, 2, 3, 5, 7})
      for (int ct : {64 / tr, 32 / tr}) {
        // The tiles that are compiled, with registers for two wavefronts a SIMD.  (Larger ones read less LDS, but one wavefront
        // a SIMD waits alone: 300C2 of 512 images in 128 x 256 694 us of the pass, in 64 x 256 543.)
        if (tr == 32 ? rt > 2 : rt == 2 || (rt > 3 && ct > 2)) continue;
        const int rows = rt * tr, cols = 4 * ct * tr, S = tr == 32 ? 2 : 4, groups = (t.Mo + rows - 1) / rows;
        if (M > cols || cols / M * M * 4 < cols * 3 || (groups > 1 && groups * rows - t.Mo >= rows / 2)) continue;
        t.RT = rt; t.CT = ct; t.TR = tr;
        t.wins = cols / M;
        // whole images, or whole rows of windows, where that leaves few columns empty: fewer pixels to stage
        if (t.wins > t.win_img && t.wins % t.win_img * 12 <= t.wins) t.wins -= t.wins % t.win_img;
        else if (t.wins > t.Wp && t.wins % t.Wp * 24 <= t.wins) t.wins -= t.wins % t.Wp;
        t.run_px = (pixels(t.wins) + 63) / 64 * 64;
        const size_t n_cb = (batch * t.win_img + t.wins - 1) / t.wins;
        for (int ic = 1; ic <= t.n_cg; ++ic) {
          if (t.n_cg % ic) continue;
          t.IC = ic;
          t.cps = t.n_cg / ic;
          t.n_kg = (ic * KK + S - 1) / S * S;
          for (int part = 1; part <= 8; ++part) {   // slabs of a chunk
            t.slab = ((t.n_kg + part - 1) / part + S - 1) / S * S;
            if (part > 1 && t.slab < 2 * S) break;
            const size_t lds = batch_split_lds_bytes(t);
            if (lds > LDS) continue;
            const double est = split_clocks(t, n_cb);
            if (best == 0 || est < best) { best = est; out = t; }
          }
        }
      }
  if (out.slab > SPLIT_RUN) {   // (a running sum is a slab at least)
    const int S = out.TR == 32 ? 2 : 4, parts = (out.n_kg + SPLIT_RUN - 1) / SPLIT_RUN;
    out.slab = ((out.n_kg + parts - 1) / parts + S - 1) / S * S;
  }
  if (out.RT) { out.by_win_img = fast_div_of(out.win_img); out.by_wp = fast_div_of(out.Wp); }
  return best;
}

// (group of maps, tap) pairs of a row that a workgroup of k_batch_pack turns into halves at a time.  Every piece of a row reads
// the whole row for its scale.
int split_piece(const BatchSplit& t) {
  const int rows = t.RT * t.TR, tiles = (t.Mo + rows - 1) / rows * rows / 4, total = t.n_cg / t.IC * t.n_kg, pieces = std::max(1, 512 / tiles);
  return std::max(128, (total + pieces - 1) / pieces);
}

// The plan of k_batch_split for a fully connected layer behind a layer of `maps` maps of `pix` pixels: as split_plan, and slices of
// the k range, at most as many as the 32-bit product has.
double fc_plan(const LayerDev& L, int maps, int pix, size_t batch, int most_slices, BatchSplit& out) {
  constexpr size_t LDS = 160 * 1024;
  BatchSplit t;
  std::memset(&t, 0, sizeof(t));
  out = t;
  t.fc = 1; t.n_cg = (maps + 7) / 8 * pix; t.pix = pix; t.by_pix = fast_div_of(pix); t.Wi = t.K = t.Kx = t.stride = t.stride_x = 1;
  t.Mo = L.n_out; t.Kp = t.Kpx = t.Wp = t.win_img = 1; t.bias = L.bias;
  const size_t limit = (size_t)1 << 29, in_floats = (size_t)t.n_cg * 8;
  // (weights that the L2 caches do not hold are read from memory once more for every piece: 600 rows of 134480 took 1.4 times as long)
  if (L.is_output || (size_t)L.n_out * maps * pix > (size_t)1 << 23 || batch * in_floats >= limit || batch * (size_t)(L.n_out + 7) >= limit) return 0;
  t.in_plane = (long long)batch * pix * 16;
  t.slice_stride = (long long)(batch * (size_t)L.n_out);
  double best = 0;
  for (int tr : {32, 16})
    for (int rt : {1, 2, 3, 5, 7})
      for (int ct : {64 / tr, 32 / tr}) {
        if (tr == 32 ? rt > 2 : rt == 2 || (rt > 3 && ct > 2)) continue;
        const int rows = rt * tr, cols = 4 * ct * tr, S = tr == 32 ? 2 : 4, groups = (t.Mo + rows - 1) / rows;
        if (groups > 1 && groups * rows - t.Mo >= rows / 2) continue;
        t.RT = rt; t.CT = ct; t.TR = tr; t.wins = t.run_px = cols;
        const size_t n_cb = (batch + cols - 1) / cols;
        for (int ic = 1; ic <= std::min(t.n_cg, SPLIT_RUN); ++ic) {   // (a chunk is a slab)
          if (t.n_cg % ic) continue;
          t.IC = ic;
          t.n_kg = t.slab = (ic + S - 1) / S * S;
          if (batch_split_lds_bytes(t) > LDS) break;
          const int chunks = t.n_cg / ic;
          for (int slices = 1; slices <= std::min(most_slices, chunks); slices *= 2) {
            t.cps = (chunks + slices - 1) / slices;
            t.raw = (chunks + t.cps - 1) / t.cps > 1;
            const double est = split_clocks(t, n_cb) + (t.raw ? 1500.0 : 0.0);
            if (best == 0 || est < best) { best = est; out = t; }
          }
        }
      }
  if (out.RT == 0) return 0;
  out.by_win_img = out.by_wp = fast_div_of(1);
  const int total = out.n_cg / out.IC * out.n_kg, piece = split_piece(out);
  return best + 4.0 * L.n_out * maps * pix * ((total + piece - 1) / piece) / 1200.0;   // (a row is read once a piece)
}

// The plan of k_batch_first for the first layer, and its clocks of a compute unit: the vector instructions of all windows (the
// products of halves run beside them), or the chain of one wavefront's members.  Leaves out.T = 0 where a sum has more terms
// than the kernel is compiled for.
double first_plan(const LayerDev& L, size_t batch, BatchFirst& out) {
  BatchFirst f;
  std::memset(&f, 0, sizeof(f));
  out = f;
  f.Hi = L.Hi; f.Wi = L.Wi; f.K = L.K; f.Kx = L.Kx; f.stride = L.S + 1; f.stride_x = L.Sx + 1; f.Mo = L.Mo;
  f.Kp = L.Kp; f.Kpx = L.Kpx; f.Wp = L.Wp; f.win_img = L.Hp * L.Wp; f.bias = L.bias;
  f.by_win_img = fast_div_of(f.win_img); f.by_wp = fast_div_of(f.Wp); f.by_kpx = fast_div_of(f.Kpx);
  f.k_total = L.Mi * L.K * L.Kx;
  f.row = (L.Mo + 15) / 16 * 16;
  if ((long long)L.Mi * L.Hi * L.Wi * 33 * 4 >= 1ll << 31) return 0;   // (32-bit offsets from the first of 32 windows)
  f.H = batch_first_steps(f.k_total);
  if (!f.H) return 0;
  const double jobs = (double)((batch * f.win_img + 31) / 32);
  const int M = L.Kp * L.Kpx;
  double best = 0;
  for (int T : {5, 2, 1})
    for (int share = 0; share < (M >= 4 && T <= 2 ? 2 : 1); ++share) {
      if ((T == 5 && f.H > 2) || (T == 2 && f.H > 5)) continue;   // (the registers)
      f.T = T; f.share = share;
      const int groups = (L.Mo + T * 32 - 1) / (T * 32);
      const double pixels = f.H * 800.0 + 150.0, sums = T * (f.H * 50.0 + 130.0), outputs = std::min(T * 32, L.Mo) * 75.0 + 300.0;
      const double all = jobs * groups * (M * (pixels + sums) + outputs) / 1024;
      const double chain = share ? (M + 3) / 4 * (pixels + sums + 1200.0) + outputs / 4 + 1500.0 : M * (pixels + sums + 1200.0) + outputs;
      const double est = 4000.0 + f.H * 300.0 + std::max(all, chain);
      if (best == 0 || est < best) { best = est; out = f; }
    }
  // A last group of maps takes eight more, from the one in front of it, where it would have eight or fewer.  One or two maps of a
  // pixel are below SPLIT_TINY by chance (with weights up to 0.05 one in 3000 of a map's activations), and every such pixel makes
  // the blocks behind that read it take 32-bit products.  424 images of 3x32x32-65C5-MP2-32C5-MP2-24C4-MP2 281 us a call, 465 with a last
  // group of one map; 143 of 2x96x96-193C6S1-MP2-217C4-MP4 593 and 1265.
  if (out.T && L.Mo > out.T * 32 && (L.Mo - 1) % (out.T * 32) < 8) out.shift = 8;
  return best;
}

// The buffer of a layer that writes halves of `eights` groups of eight maps of `pix` pixels for `s`: the halves, and their marks.
void marked(BatchStep& below, BatchSplit& s, size_t eights, size_t pix) {
  const int rows = below.f.T ? below.f.T * 32 : below.s.RT * below.s.TR;
  s.in_shift = below.f.T ? below.f.shift / 8 : 0;
  s.in_groups = (int)(((eights + s.in_shift) * 8 + rows - 1) / rows);
  s.by_eights = fast_div_of(rows / 8);
  below.halves_per_image = eights * 8 * pix;
  below.out_per_image = below.halves_per_image + (s.in_groups * pix + 3) / 4;
}

// Shape of every layer's matrix product, tile choice and LDS budget.  Returns 0 or an error code.  split: convolutional layers
// behind another one in products of halves, where their plan fits.
int batch_plan_of(cnn* net, size_t batch, bool split, BatchPlan& B) {
  const ProgramDev& P = net->prog;
  constexpr size_t LDS_FLOATS = 20000;      // 78 KB per workgroup: two workgroups per compute unit
  constexpr size_t LDS_FLOATS_BIG = 38000;  // large input maps: one workgroup per compute unit
  B = BatchPlan();
  for (int l = 0; l < P.n_layers; ++l) {
    const LayerDev& L = P.layers[l];
    BatchStep st;
    BatchGemm& g = st.g;
    std::memset(&g, 0, sizeof(g));
    int Kp = 1, Kpx = 1, Ho = 1, Hp = 1, Wp = 1;
    if (L.kind == L_CONV) {
      g.Mi = L.Mi; g.Hi = L.Hi; g.Wi = L.Wi; g.K = L.K; g.Kx = L.Kx; g.stride = L.S + 1; g.stride_x = L.Sx + 1;
      g.Mo = L.Mo; g.Wo = L.Wo;
      g.P = L.Ho * L.Wo; Ho = L.Ho; Kp = L.Kp; Kpx = L.Kpx; Hp = L.Hp; Wp = L.Wp;
    } else {  // a fully connected layer: n_in maps of one pixel, K = 1
      g.Mi = L.n_in; g.Hi = 1; g.Wi = 1; g.K = 1; g.Kx = 1; g.stride = 1; g.stride_x = 1; g.Mo = L.n_out; g.Wo = 1; g.P = 1;
    }
    const bool pooled = Kp * Kpx > 1;
    // map tiles per workgroup: the choice that pads the fewest maps, the larger on a tie; tiles of 16 maps only
    // where they pad fewer than tiles of 32 do (40 maps: 48 rows instead of 64), at least two of them a workgroup
    // (an operand fetched from the staged images should feed several instructions)
    int best_pad = 0;
    g.TR = 32;
    for (int mt : {4, 2, 1}) {
      const int pad = (g.Mo + 32 * mt - 1) / (32 * mt) * (32 * mt);
      if (!best_pad || pad < best_pad) { best_pad = pad; g.MT = mt; }
    }
    for (int mt : {6, 5, 4, 3, 2}) {
      const int pad = (g.Mo + 16 * mt - 1) / (16 * mt) * (16 * mt);
      if (pad < best_pad) { best_pad = pad; g.MT = mt; g.TR = 16; }
    }
    g.MoPad = best_pad;
    const int KK = g.K * g.Kx, HiWi = g.Hi * g.Wi;
    // input maps per chunk: as many as the LDS budget takes; when that leaves several chunks,
    // prefer a chunk that also fits the prefetch registers (16 + 48 floats per thread), unless
    // such a chunk would be too short to hide anything behind.  One-pixel maps (fully connected
    // layers) take a power of two, so that staging finds image and offset by shifting.
    int ic = 0, ic_pre = 0;
    auto fit = [&](int cols_per_image, size_t budget) {
      g.n_img_max = (int)std::min<size_t>(std::max<size_t>(batch, 1), (size_t)((128 - 1 + cols_per_image - 1) / cols_per_image + 1));
      ic = 0; ic_pre = 0;
      for (int c = 1; c <= g.Mi; ++c) {
        const size_t in_f = (size_t)g.n_img_max * c * HiWi, w_f = (size_t)(c * KK + 1) * g.MT * g.TR;
        if (in_f + 3 + w_f + (size_t)c * KK + (g.TR == 32 ? 9 : 20) > budget) break;
        if (HiWi == 1 && c < g.Mi && (c & (c - 1)) != 0) continue;
        ic = c;
        if (in_f <= 16 * 256 && w_f <= 48 * 256) ic_pre = c;
      }
    };
    // Pooling inside the product: when the whole k range is one chunk, a column is a pooled pixel
    // and the wavefront walks the Kp x Kpx members of its window one after the other, keeping the
    // running maximum in registers; the full-resolution sums then never reach memory.
    g.Kp = 1; g.Kpx = 1;
    bool pool_inside = false;
    if (pooled) {
      fit(Hp * Wp, LDS_FLOATS);
      if (ic == g.Mi) { g.Kp = Kp; g.Kpx = Kpx; g.P = Hp * Wp; g.Wo = Wp; pool_inside = true; }
    }
    if (!pool_inside) {
      fit(g.P, LDS_FLOATS);
      if (ic == 0) fit(g.P, LDS_FLOATS_BIG);
    }
    if (ic == 0)
      return fail(&net->err, CNN_E_SHAPE, "batched forward pass: one input map of a layer (times the images a "
                                          "workgroup touches) exceeds the LDS budget");
    g.prefetch = 0;
    if (ic < g.Mi && ic_pre * KK >= 96) { ic = ic_pre; g.prefetch = 1; }
    g.IC = ic;
    // few columns and a long k range (fully connected layers, deep layers on small maps): the k
    // range is cut into slices, one workgroup each, until some 512 workgroups are in flight
    const int n_chunks = (g.Mi + ic - 1) / ic;
    const size_t wgs = ((batch * g.P + 127) / 128) * (size_t)(g.MoPad / (g.TR * g.MT));
    int ks = 1;
    if (wgs < 512 && n_chunks > 1) ks = (int)std::min<size_t>((size_t)n_chunks, (512 + wgs - 1) / wgs);
    g.chunks_per_slice = (n_chunks + ks - 1) / ks;
    g.KS = (n_chunks + g.chunks_per_slice - 1) / g.chunks_per_slice;
    g.slice_stride = (long long)(batch * g.Mo * g.P);
    g.fuse = ((pooled && !pool_inside) || g.KS > 1) ? 0 : (L.is_output ? 2 : 1);
    g.bias = L.bias;
    g.in_stride = (long long)g.Mi * HiWi;
    g.out_stride = (long long)g.Mo * g.P;
    std::memset(&st.c, 0, sizeof(st.c));
    if (L.kind == L_CONV) conv_plan(L, g, batch, st.c);
    const BatchConv& c = st.c;
    int KSl = c.MT ? c.n_slices : g.KS;
    std::memset(&st.s, 0, sizeof(st.s));
    std::memset(&st.f, 0, sizeof(st.f));
    auto old_clocks = [&](const BatchStep& t) {
      return t.c.MT ? conv_clocks(t.c, batch, (batch * t.c.win_img + t.c.wins - 1) / t.c.wins) : gemm_clocks(t.g, batch);
    };
    if (split && L.kind == L_CONV && l > 0 && P.layers[l - 1].kind == L_CONV && (B.steps.back().s.RT || l == 1)) {
      BatchStep& below = B.steps.back();
      double est = split_plan(L, batch, st.s), old = old_clocks(st);
      const bool with_first = !below.s.RT;
      if (st.s.RT && with_first) {   // the first layer comes with it
        est += first_plan(P.layers[0], batch, below.f);
        old += old_clocks(below);
        if (!below.f.T) st.s.RT = 0;
      }
      // where that is the faster form: over 216 nets of 1 to 10000 images 8 lose by it, 31 us of 14 ms together, and 6 that would
      // gain 31 us are left as they were
      if (0.8 * est + (with_first ? 8000.0 : 2000.0) >= old) st.s.RT = 0;
      if (st.s.RT) {
        below.split_out = true;
        marked(below, st.s, (size_t)st.s.n_cg, (size_t)HiWi);
        (below.s.RT ? below.s.split_out : below.f.split_out) = (int)(batch * (size_t)HiWi);
        if (below.f.T) {
          B.wt_total -= below.wt_floats;
          below.wt_floats = up64((size_t)below.f.k_total * below.f.row);
          B.wt_total += below.wt_floats;
          below.pack.row = below.f.row;
        }
      } else {
        below.f.T = 0;
      }
    }
    if (split && L.kind != L_CONV && l > 0 && B.steps.back().s.RT) {
      BatchStep& below = B.steps.back();
      const LayerDev& prev = P.layers[l - 1];
      const int maps = prev.kind == L_CONV ? prev.Mo : prev.n_out, pix = prev.kind == L_CONV ? prev.Hp * prev.Wp : 1;
      const double est = below.raw() ? 0.0 : fc_plan(L, maps, pix, batch, g.KS, st.s);
      if (st.s.RT == 0 || 0.8 * est + 2000.0 >= gemm_clocks(g, batch)) std::memset(&st.s, 0, sizeof(st.s));
      else {
        st.s.drop = g.fuse == 0;
        below.split_out = true;
        marked(below, st.s, (size_t)st.s.n_cg / pix, (size_t)pix);
        below.s.split_out = (int)(batch * (size_t)pix);
      }
    }
    const BatchSplit& h = st.s;
    const int h_rows = h.RT * h.TR, h_groups = h.RT ? (h.Mo + h_rows - 1) / h_rows : 0;
    st.wt_floats = h.RT ? up64((size_t)h_groups * h_rows * (h.n_cg / h.IC) * h.n_kg * 8) + up64((size_t)h_groups * h_rows + 1) : up64((size_t)g.Mi * KK * (c.MT ? (size_t)(c.Mo + c.MT * c.TR - 1) / (c.MT * c.TR) * (c.MT * c.TR) : (size_t)g.MoPad));
    st.wt_off = B.wt_total;
    B.wt_total += st.wt_floats;
    BatchPack& k = st.pack;
    std::memset(&k, 0, sizeof(k));
    k.w = L.w; k.csr_ptr = L.csr_ptr; k.csr_idx = L.csr_idx;
    k.full_table = L.kind != L_CONV || L.full_table; k.Mo = g.Mo; k.K = g.K; k.Kx = g.Kx;
    k.row = h.RT ? h_rows : c.MT ? c.MT * c.TR : g.MoPad; k.k_total = g.Mi * KK;
    k.Mi = g.Mi; k.n_chunks = h.RT ? h.n_cg / h.IC : 0; k.n_kg = h.n_kg; k.piece = h.RT ? split_piece(h) : 0; k.per_chunk = h.fc ? h.IC : h.IC * KK;
    if (h.fc) {   // inputs are (map, pixel): a map's pixels are the taps of its kernel
      const LayerDev& prev = P.layers[l - 1];
      k.Mi = prev.kind == L_CONV ? prev.Mo : prev.n_out;
      k.K = prev.kind == L_CONV ? prev.Hp : 1; k.Kx = prev.kind == L_CONV ? prev.Wp : 1;
    }
    if (h.RT) KSl = (h.n_cg / h.IC + h.cps - 1) / h.cps;
    BatchPool& q = st.pool;
    std::memset(&q, 0, sizeof(q));
    q.bias = L.bias; q.Mo = g.Mo; q.Ho = Ho; q.Wo = (L.kind == L_CONV) ? L.Wo : 1; q.Kp = Kp; q.Kpx = Kpx; q.Hp = Hp; q.Wp = Wp;
    q.n_slices = KSl; q.slice_stride = c.MT ? (long long)(batch * L.Mo * L.Ho * L.Wo) : g.slice_stride; q.act = L.is_output ? 0 : 1;
    st.out_per_image = pooled ? (size_t)g.Mo * Hp * Wp : (size_t)g.Mo * g.P;
    if (c.MT) { st.c.slice_stride = q.slice_stride; st.c.out_stride = (long long)c.Mo * c.win_img; }
    if (h.RT) st.s.out_stride = (long long)st.out_per_image;
    if (h.fc) q.slice_stride = h.slice_stride;
    if (st.raw()) B.sums_per_image = std::max(B.sums_per_image, up64((size_t)KSl * g.Mo * (c.MT ? c.win_img : g.P)));
    // (the columns are the layer's pixels whenever fuse == 0 with pooling: pooling inside the product has fuse != 0)
    B.steps.push_back(st);
  }
  if (P.n_layers > 1 && P.layers[P.n_layers - 2].kind != L_CONV) {
    const LayerDev &hidden = P.layers[P.n_layers - 2], &out = P.layers[P.n_layers - 1];
    B.tail = out.is_output && out.kind != L_CONV && hidden.n_out <= TAIL_HIDDEN && out.n_out <= TAIL_OUT && hidden.n_out * out.n_out <= TAIL_WEIGHTS;
  }
  size_t act[2] = {0, 0};
  bool any = false;
  for (size_t l = 0; l < B.steps.size(); ++l) {
    act[l & 1] = std::max(act[l & 1], up64(B.steps[l].out_per_image));
    any |= B.steps[l].split_out;
  }
  // (two buffers of the same size where every product is one of 32 bits)
  for (size_t l = 0; l < 2; ++l) B.act_per_image[l] = any ? act[l] : std::max(act[0], act[1]);
  if (P.has_frontend) B.fe_per_image = up64((size_t)P.fe.n_filters * P.fe.H * P.fe.W);
  return CNN_OK;
}

// Products of halves, unless the maps that fill groups of eight and tiles up take more scratch memory than 32-bit products
// throughout: a caller whose memory was enough for a batch goes on with it.  The caller is asked for what the latter take:
// fewer images may run in 32-bit products where more run in halves (60 digits 1 M floats, 100 digits 0.6 M), and a program
// with memory for its batch calls with what remains of a set.
int batch_plan(cnn* net, size_t batch, BatchPlan& B) {
  const int rc = batch_plan_of(net, batch, false, B);
  if (rc) return rc;
  const size_t asked = B.floats(batch);
  BatchPlan halves;
  if (batch_plan_of(net, batch, true, halves) == CNN_OK && halves.floats(batch) <= asked) B = std::move(halves);
  B.asked = asked;
  return CNN_OK;
}

// The plan of a handle for a batch.  The last few are kept, with all that they were made from, and taken again while that is the
// same: making one takes 9 to 58 us of the host's time (2.7 to 14 for 32-bit products alone), which a single call waits for.  Few,
// and not one: a program goes back and forth between batches (training and validation sets, what remains of one), or asks for
// another one's memory in between.  The lock is for calls that ask for memory side by side: they only read the handle otherwise.
constexpr size_t BATCH_KEPT = 4;
int batch_plan(cnn* net, size_t batch, std::shared_ptr<const BatchKept>& out);

}  // namespace

struct BatchKept {
  size_t batch;
  int has_frontend, n_filters, fe_h, fe_w;
  std::vector<LayerDev> layers;
  BatchPlan plan;
  bool made_for(const ProgramDev& P, size_t n) const {
    return n == batch && P.has_frontend == has_frontend && P.fe.n_filters == n_filters && P.fe.H == fe_h && P.fe.W == fe_w &&
           (size_t)P.n_layers == layers.size() && std::memcmp(layers.data(), P.layers, layers.size() * sizeof(LayerDev)) == 0;
  }
};

namespace {
int batch_plan(cnn* net, size_t batch, std::shared_ptr<const BatchKept>& out) {
  const ProgramDev& P = net->prog;
  std::lock_guard<std::mutex> hold(net->batch_kept_lock);
  auto& kept = net->batch_kept;
  size_t at = 0;
  while (at < kept.size() && !kept[at]->made_for(P, batch)) ++at;
  if (at == kept.size()) {
    auto made = std::make_shared<BatchKept>();
    const int rc = batch_plan(net, batch, made->plan);
    if (rc) return rc;
    made->batch = batch;
    made->has_frontend = P.has_frontend; made->n_filters = P.fe.n_filters; made->fe_h = P.fe.H; made->fe_w = P.fe.W;
    made->layers.assign(P.layers, P.layers + P.n_layers);
    if (kept.size() < BATCH_KEPT) kept.push_back(nullptr);
    at = kept.size() - 1;
    kept[at] = std::move(made);
  }
  std::rotate(kept.begin(), kept.begin() + at, kept.begin() + at + 1);
  out = kept.front();
  return CNN_OK;
}
}  // namespace

extern "C" {

int cnn_arch_info(const char* arch, int32_t* n_layers, int32_t* info, int32_t max_layers) {
  std::vector<ArchLayer> A;
  int rc = parse_arch(arch, A, nullptr);
  if (rc) return rc;
  if (n_layers) *n_layers = (int32_t)A.size();
  if (info)
    for (size_t l = 0; l < A.size() && (int32_t)l < max_layers; ++l) {
      int32_t* o = info + 6 * l;
      o[0] = A[l].kind; o[1] = A[l].maps; o[2] = A[l].h; o[3] = A[l].w; o[4] = A[l].K; o[5] = A[l].S;
    }
  return CNN_OK;
}

int cnn_arch_info_xy(const char* arch, int32_t* n_layers, int32_t* info, int32_t max_layers) {
  std::vector<ArchLayer> A;
  int rc = parse_arch(arch, A, nullptr);
  if (rc) return rc;
  if (n_layers) *n_layers = (int32_t)A.size();
  if (info)
    for (size_t l = 0; l < A.size() && (int32_t)l < max_layers; ++l) {
      int32_t* o = info + 8 * l;
      o[0] = A[l].kind; o[1] = A[l].maps; o[2] = A[l].h; o[3] = A[l].w; o[4] = A[l].K; o[5] = A[l].S;
      o[6] = A[l].Kx; o[7] = A[l].Sx;
    }
  return CNN_OK;
}

int cnn_workspace_bytes(const char* arch, size_t* bytes) {
  if (!bytes) return fail(nullptr, CNN_E_ARG, "bytes is NULL");
  cnn tmp;
  int rc = parse_arch(arch, tmp.arch, nullptr);
  if (rc) return rc;
  *bytes = carve(&tmp, nullptr);
  for (size_t l = 1; l < tmp.arch.size(); ++l)
    if (tmp.arch[l].kind == CNN_LAYER_CONV)
      tmp.tables.emplace_back((size_t)tmp.arch[l].maps * tmp.arch[l - 1].maps, (uint8_t)1);
  rc = plan(&tmp);  // shapes the kernels cannot take are refused here, without a device
  if (rc) g_err = tmp.err;
  return rc;
}

static int plan_to_text(const ProgramDev& P, char* buf, size_t n) {
  static const char* names[] = {"?", "frontend", "conv_fwd", "fc_fwd", "head", "fc_bwd", "conv_bwd", "conv_wgrad", "conv_mfma", "conv_epi",
                                "conv_bwd_mfma", "conv_bwd_epi", "conv_wgrad_mfma", "conv_wgrad_win", "conv_bwd_win", "conv_bwd_wepi", "conv_fwd_mx", "conv_wgrad_first"};
  std::string out;
  char line[256];
  for (int s = 0; s < P.n_stages; ++s) {
    const Stage& st = P.stages[s];
    std::snprintf(line, sizeof line, "%2d %-10s layer=%d items=%d barrier=%d train_only=%d rows=%d tiles=%d chunk=%d tw=%d ppt=%d rpw=%d cm=%d\n",
                  s, names[st.kind], st.layer, st.n_items, st.barrier_after, st.train_only, st.tile_rows, st.n_tiles,
                  st.chunk, 1 << st.tw_log2, st.pix_per_thread, st.rows_per_wg, 1 << st.cm_log2);
    out += line;
  }
  std::snprintf(buf, n, "%s", out.c_str());
  return CNN_OK;
}

int cnn_plan_text(const char* arch, char* buf, size_t n) {
  if (!buf || n == 0) return fail(nullptr, CNN_E_ARG, "buf is NULL");
  cnn tmp;
  int rc = parse_arch(arch, tmp.arch, nullptr);
  if (rc) return rc;
  carve(&tmp, nullptr);
  for (size_t l = 1; l < tmp.arch.size(); ++l)
    if (tmp.arch[l].kind == CNN_LAYER_CONV)
      tmp.tables.emplace_back((size_t)tmp.arch[l].maps * tmp.arch[l - 1].maps, (uint8_t)1);
  rc = plan(&tmp);
  if (rc) { g_err = tmp.err; return rc; }
  return plan_to_text(tmp.prog, buf, n);
}

int cnn_get_plan_text(const cnn_t* net, char* buf, size_t n) {
  if (!net || !buf || n == 0) return CNN_E_ARG;
  return plan_to_text(net->prog, buf, n);
}

int cnn_create(const char* arch, void* d_workspace, size_t bytes, void* hip_stream, cnn_t** out) {
  if (!out) return fail(nullptr, CNN_E_ARG, "out is NULL");
  *out = nullptr;
  cnn* net = new cnn;
  int rc = parse_arch(arch, net->arch, &net->err);
  if (rc) { delete net; return rc; }
  const size_t need = carve(net, nullptr);
  if (!d_workspace || bytes < need || ((uintptr_t)d_workspace & 255)) {
    delete net;
    return fail(nullptr, CNN_E_WORKSPACE, "workspace must be 256-byte aligned device memory of at least " +
                                              std::to_string(need) + " bytes");
  }
  carve(net, d_workspace);
  net->stream = (hipStream_t)hip_stream;
  for (size_t l = 1; l < net->arch.size(); ++l)
    if (net->arch[l].kind == CNN_LAYER_CONV)
      net->tables.emplace_back((size_t)net->arch[l].maps * net->arch[l - 1].maps, (uint8_t)1);
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&net->n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&net->coop_ok, hipDeviceAttributeCooperativeLaunch, dev);
  if (e != hipSuccess) { rc = hip_fail(nullptr, e, "device query"); delete net; return rc; }
  net->device = dev;
  net->max_blocks_per_cu = std::max(1, persistent_max_blocks_per_cu());
  rc = rebuild(net);
  if (rc) { g_err = net->err; delete net; return rc; }
  *out = net;
  return CNN_OK;
}

void cnn_destroy(cnn_t* net) {
  if (!net) return;
  (void)hipStreamSynchronize(net->stream);
  if (net->special_module) (void)hipModuleUnload(net->special_module);
  drop_stage_graphs(net);
  delete net;
}

int cnn_set_connection_table(cnn_t* net, int conv_index, const uint8_t* host_table) {
  if (!net || !host_table) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (conv_index < 0 || conv_index >= (int)net->tables.size()) return fail(&net->err, CNN_E_ARG, "no such convolutional layer");
  int seen = 0, mo = 0, mi = 0;
  for (size_t l = 1; l < net->arch.size(); ++l)
    if (net->arch[l].kind == CNN_LAYER_CONV && seen++ == conv_index) { mo = net->arch[l].maps; mi = net->arch[l - 1].maps; }
  std::vector<uint8_t> t((size_t)mo * mi);
  for (int j = 0; j < mo; ++j) {
    bool any = false;
    for (int i = 0; i < mi; ++i) { t[(size_t)j * mi + i] = host_table[(size_t)j * mi + i] ? 1 : 0; any |= t[(size_t)j * mi + i] != 0; }
    if (!any) return fail(&net->err, CNN_E_ARG, "output map " + std::to_string(j) + " has no input map");
  }
  net->tables[conv_index] = t;
  return rebuild(net);
}

int cnn_set_fixed_frontend(cnn_t* net, int n_filters, int K, int n_src_channels, const float* host_filters,
                           const int32_t* host_src_channel) {
  if (!net || !host_filters || !host_src_channel) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (n_filters != net->arch[0].maps) return fail(&net->err, CNN_E_ARG, "n_filters must equal the input maps of the architecture");
  if (K < 1 || K > MAX_FRONTEND_K || n_src_channels < 1) return fail(&net->err, CNN_E_ARG, "bad front-end size");
  for (int f = 0; f < n_filters; ++f)
    if (host_src_channel[f] < 0 || host_src_channel[f] >= n_src_channels) return fail(&net->err, CNN_E_ARG, "source channel out of range");
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  net->fe_n = n_filters; net->fe_K = K; net->fe_src_n = n_src_channels;
  net->fe_filters.assign(host_filters, host_filters + (size_t)n_filters * K * K);
  net->fe_src.assign(host_src_channel, host_src_channel + n_filters);
  HIP_TRY(net, hipMemcpy(net->d_fe_filters, net->fe_filters.data(), net->fe_filters.size() * 4, hipMemcpyHostToDevice));
  HIP_TRY(net, hipMemcpy(net->d_fe_src, net->fe_src.data(), net->fe_src.size() * 4, hipMemcpyHostToDevice));
  return rebuild(net);
}

size_t cnn_num_weights(const cnn_t* net) { return net ? net->n_weights : 0; }
size_t cnn_image_size(const cnn_t* net) { return net ? net->image_size : 0; }
int cnn_num_layers(const cnn_t* net) { return net ? (int)net->arch.size() : 0; }
int cnn_num_classes(const cnn_t* net) { return net ? net->n_classes : 0; }

int cnn_layer_info(const cnn_t* net, int layer, int32_t* o) {
  if (!net || !o || layer < 0 || layer >= (int)net->arch.size()) return CNN_E_ARG;
  const ArchLayer& a = net->arch[layer];
  o[0] = a.kind; o[1] = a.maps; o[2] = a.h; o[3] = a.w; o[4] = a.K; o[5] = a.S;
  return CNN_OK;
}

int cnn_layer_info_xy(const cnn_t* net, int layer, int32_t* o) {
  if (!net || !o || layer < 0 || layer >= (int)net->arch.size()) return CNN_E_ARG;
  const ArchLayer& a = net->arch[layer];
  o[0] = a.kind; o[1] = a.maps; o[2] = a.h; o[3] = a.w; o[4] = a.K; o[5] = a.S; o[6] = a.Kx; o[7] = a.Sx;
  return CNN_OK;
}

int cnn_get_weights(cnn_t* net, float* host_dst, size_t n) {
  if (!net || !host_dst) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (n != net->n_weights) return fail(&net->err, CNN_E_ARG, "weight count mismatch");
  int rc = sync_and_check(net);
  HIP_TRY(net, hipMemcpy(host_dst, net->d_weights, n * sizeof(float), hipMemcpyDeviceToHost));
  return rc;
}

int cnn_set_weights(cnn_t* net, const float* host_src, size_t n) {
  if (!net || !host_src) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (n != net->n_weights) return fail(&net->err, CNN_E_ARG, "weight count mismatch");
  int rc = sync_and_check(net);
  HIP_TRY(net, hipMemcpy(net->d_weights, host_src, n * sizeof(float), hipMemcpyHostToDevice));
  return rc;
}

int cnn_forward(cnn_t* net, const float* d_image, float* d_probs) {
  return cnn_forward_many(net, d_image, 1, d_probs);
}

int cnn_forward_many(cnn_t* net, const float* d_images, size_t n, float* d_probs) {
  if (!net || !d_images) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (n == 0) return CNN_OK;
  RunArgs a;
  std::memset(&a, 0, sizeof(a));
  a.images = d_images; a.probs_out = d_probs; a.n_images = (long long)n; a.image_stride = (long long)net->image_size;
  a.label_imm = -1; a.train = 0;
  return run(net, a);
}

int cnn_train_step(cnn_t* net, const float* d_image, int32_t label, float lr) {
  if (!net || !d_image) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (label < 0 || label >= net->n_classes) return fail(&net->err, CNN_E_ARG, "label out of range");
  RunArgs a;
  std::memset(&a, 0, sizeof(a));
  a.images = d_image; a.n_images = 1; a.image_stride = (long long)net->image_size;
  a.label_imm = label; a.train = 1; a.lr = lr;
  return run(net, a);
}

int cnn_train_many(cnn_t* net, const float* d_images, const int32_t* d_labels, size_t n, float lr) {
  if (!net || !d_images || !d_labels) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (n == 0) return CNN_OK;
  RunArgs a;
  std::memset(&a, 0, sizeof(a));
  a.images = d_images; a.labels = d_labels; a.n_images = (long long)n; a.image_stride = (long long)net->image_size;
  a.train = 1; a.lr = lr;
  return run(net, a);
}

int cnn_set_mode(cnn_t* net, int mode) {
  if (!net) return CNN_E_ARG;
  if (mode != CNN_MODE_STAGES && mode != CNN_MODE_PERSISTENT && mode != CNN_MODE_RESIDENT)
    return fail(&net->err, CNN_E_ARG, "unknown mode");
  if (mode != CNN_MODE_STAGES && !net->coop_ok) return fail(&net->err, CNN_E_STATE, "device does not support cooperative launches");
  if (mode == CNN_MODE_RESIDENT && !net->flow_ok) return fail(&net->err, CNN_E_STATE, net->flow_why);
  // every mode has a stage list of its own: the pull and the gradients over the winners and the matrix-core pull are
  // planned for the stage launches only, the first layer's matrix-core product for all but the persistent kernel
  return mode == net->mode ? CNN_OK : replan(net, mode);
}

int cnn_mode_supported(cnn_t* net, int mode) {
  if (!net) return 0;
  if (mode == CNN_MODE_STAGES) return 1;
  if (mode == CNN_MODE_PERSISTENT) return net->coop_ok ? 1 : 0;
  if (mode == CNN_MODE_RESIDENT) return (net->coop_ok && net->flow_ok) ? 1 : 0;
  return 0;
}

int cnn_get_mode(const cnn_t* net) { return net ? net->mode : CNN_E_ARG; }

// ---- a resident kernel compiled for the handle's own network -----------------------------------------
// The text of a header that gives cnn355_flowspec.h the network of this handle as StaticSpec<FLOW_SPECIAL_ID>:
// the same inputs plan_flow() hands the planner, so the compiler arrives at the same plan.
int cnn_resident_spec_source(const cnn_t* net, char* buf, size_t n) {
  if (!net) return fail(nullptr, CNN_E_ARG, "net is NULL");
  if (!net->flow_ok) return fail(nullptr, CNN_E_STATE, "resident mode cannot run this network: " + net->flow_why);
  const FlowSpec& Z = net->flow;
  std::string t = "// written by cnn_resident_spec_source\n";
  t += "constexpr FlowSpec flow_special_spec() {\n  FlowSpec Z{};\n";
  auto set = [&](const std::string& name, int v) { t += "  Z." + name + " = " + std::to_string(v) + ";\n"; };
  set("n_conv", Z.n_conv); set("n_fc", Z.n_fc); set("n_classes", Z.n_classes); set("out_units", Z.out_units);
  for (int l = 0; l < Z.n_conv; ++l) {
    const ConvSpec& C = Z.conv[l];
    const std::string c = "conv[" + std::to_string(l) + "].";
    set(c + "Mi", C.Mi); set(c + "Hi", C.Hi); set(c + "Wi", C.Wi); set(c + "Mo", C.Mo); set(c + "Ho", C.Ho); set(c + "Wo", C.Wo);
    set(c + "K", C.K); set(c + "S", C.S); set(c + "Kp", C.Kp); set(c + "Hp", C.Hp); set(c + "Wp", C.Wp);
    set(c + "max_conn", C.max_conn); set(c + "max_back", C.max_back); set(c + "full_table", C.full_table);
  }
  for (int f = 0; f < Z.n_fc; ++f) {
    const std::string c = "fc[" + std::to_string(f) + "].";
    set(c + "n_in", Z.fc[f].n_in); set(c + "n_out", Z.fc[f].n_out); set(c + "is_output", Z.fc[f].is_output);
  }
  t += "  flow_plan(Z, " + std::to_string(net->team_ranks) + ", " + std::to_string(net->team_stride) + ", " +
       std::to_string(net->n_cu > 0 ? net->n_cu : 256) + ");\n  return Z;\n}\n";
  t += "template <>\nstruct StaticSpec<FLOW_SPECIAL_ID> {\n  static constexpr FlowSpec value = flow_special_spec();\n};\n";
  if (buf && n > 0) {
    const size_t k = std::min(n - 1, t.size());
    std::memcpy(buf, t.data(), k);
    buf[k] = 0;
  }
  return (int)t.size();
}

int cnn_load_resident_code(cnn_t* net, const char* path) {
  if (!net || !path) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (!net->d_status) return fail(&net->err, CNN_E_STATE, "cnn_load_resident_code: the handle has no workspace");
  if (!net->flow_ok) return fail(&net->err, CNN_E_STATE, "resident mode cannot run this network: " + net->flow_why);
  int device = -1;
  HIP_TRY(net, hipGetDevice(&device));
  if (device != net->device)
    return fail(&net->err, CNN_E_STATE, "cnn_load_resident_code: the current device is not the one the network was created on");
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  hipModule_t mod = nullptr;
  if (hipModuleLoad(&mod, path) != hipSuccess) {
    (void)hipGetLastError();
    return fail(&net->err, CNN_E_ARG, std::string("cannot load a gfx950 code object from ") + path);
  }
  auto drop = [&](int code, const std::string& why) { (void)hipModuleUnload(mod); return fail(&net->err, code, why); };
  hipDeviceptr_t d_plan = nullptr;
  size_t bytes = 0;
  if (hipModuleGetGlobal(&d_plan, &bytes, mod, "cnn355_special_plan") != hipSuccess || bytes != sizeof(FlowSpec)) {
    (void)hipGetLastError();
    return drop(CNN_E_ARG, "the code object holds no plan of this library's layout (built from other sources?)");
  }
  FlowSpec plan;
  if (hipMemcpy(&plan, d_plan, sizeof(FlowSpec), hipMemcpyDeviceToHost) != hipSuccess) {
    (void)hipGetLastError();
    return drop(CNN_E_HIP, "cannot read the plan out of the code object");
  }
  if (std::memcmp(&plan, &net->flow, sizeof(FlowSpec)) != 0)
    return drop(CNN_E_STATE, "the code object was compiled for another network, table, output variant or team than this "
                             "handle has now");
  hipFunction_t f = nullptr;
  if (hipModuleGetFunction(&f, mod, "_ZN6cnn35510k_residentILi99EEEvNS_8FlowSpecEPKNS_8FlowPtrsEPNS_9StatusDevENS_7RunArgsE") != hipSuccess) {
    (void)hipGetLastError();
    return drop(CNN_E_ARG, "the code object holds no resident kernel");
  }
  if (net->special_module) (void)hipModuleUnload(net->special_module);
  net->special_module = mod;
  net->special_func = f;
  net->special_plan = plan;
  net->special_active = true;
  return CNN_OK;
}

int cnn_resident_code_active(const cnn_t* net) { return (net && net->flow_ok && net->special_active) ? 1 : 0; }

// development aid, not part of the public header: which compiled-in network the resident plan equals (0: none)
int cnn355_resident_static_id(const cnn_t* net) { return net ? net->flow_static_id : -1; }
// development aid: 1 when the resident plan streams the inputs of the layers above the first (0: they stay in LDS)
int cnn355_resident_streams(const cnn_t* net) { return (net && net->flow_ok) ? net->flow.stream : 0; }
// development aid: workgroups in the resident plan's team (0 when the network cannot run in resident mode)
int cnn355_resident_ranks(const cnn_t* net) { return (net && net->flow_ok) ? net->flow.G : 0; }
// development aid, host only (no device is touched): the resident plan of an architecture as text.  fan_in > 0
// gives every convolutional layer above the first a table in which output map j reads the input maps
// j, j + 1, ..., j + fan_in - 1 (mod M_i); fan_in = -d stands for M_i / d of them in every layer.  One line per number ("name value"), per layer ("conv l name value ...")
// and per LDS region of a rank ("region name first_float floats"); a region's size is restated here from its
// documented shape, not taken from the planner.
static int plan_only(cnn& tmp, const char* arch, int fan_in, int n_ranks, int xcd_stride) {
  int rc = parse_arch(arch, tmp.arch, nullptr);
  if (rc) return rc;
  carve(&tmp, nullptr);
  for (size_t l = 1; l < tmp.arch.size(); ++l)
    if (tmp.arch[l].kind == CNN_LAYER_CONV) {
      const int Mo = tmp.arch[l].maps, Mi = tmp.arch[l - 1].maps;
      const int fan = fan_in < 0 ? std::max(1, Mi / -fan_in) : fan_in;
      const bool sparse = fan > 0 && fan < Mi && !tmp.tables.empty();
      tmp.tables.emplace_back((size_t)Mo * Mi, (uint8_t)(sparse ? 0 : 1));
      if (sparse)
        for (int j = 0; j < Mo; ++j)
          for (int k = 0; k < fan; ++k) tmp.tables.back()[(size_t)j * Mi + (j + k) % Mi] = 1;
    }
  tmp.team_ranks = n_ranks;
  tmp.team_stride = xcd_stride;
  rc = plan(&tmp);
  if (rc) g_err = tmp.err;
  return rc;
}

// development aid, host only: cnn_resident_spec_source for an architecture without a handle (tables as in
// cnn355_resident_plan_text), so that code objects can be compiled where there is no GPU
int cnn355_resident_spec_source_for(const char* arch, int fan_in, int n_ranks, int xcd_stride, char* buf, size_t n) {
  cnn tmp;
  const int rc = plan_only(tmp, arch, fan_in, n_ranks, xcd_stride);
  if (rc) return rc;
  return cnn_resident_spec_source(&tmp, buf, n);
}

int cnn355_resident_plan_text(const char* arch, int fan_in, int n_ranks, int xcd_stride, char* buf, size_t n) {
  if (!buf || n == 0) return fail(nullptr, CNN_E_ARG, "buf is NULL");
  cnn tmp;
  int rc = plan_only(tmp, arch, fan_in, n_ranks, xcd_stride);
  if (rc) return rc;
  std::string t;
  auto num = [&](const char* name, long long v) { t += std::string(name) + " " + std::to_string(v) + "\n"; };
  if (!tmp.flow_ok) {
    t = "unsupported " + tmp.flow_why + "\n";
  } else {
    const FlowSpec& Z = tmp.flow;
    num("G", Z.G); num("stride", Z.stride); num("n_conv", Z.n_conv); num("n_fc", Z.n_fc);
    num("n_col_ranks", Z.n_col_ranks); num("fc1_owned", Z.fc1_owned); num("lds_floats", Z.lds_floats); num("lds_floats_max", FLOW_LDS_FLOATS_MAX);
    num("scratch_floats", Z.scratch_floats); num("defer", Z.defer); num("static_id", tmp.flow_static_id);
    num("stream", Z.stream);
    num("workgroup", WG); num("share_min_macs", FLOW_SHARE_MIN_MACS);
    auto region = [&](const std::string& name, long long off, long long floats) {
      t += "region " + name + " " + std::to_string(off) + " " + std::to_string(floats) + "\n";
    };
    long long act = 1, dall = 1;
    for (int l = 0; l < Z.n_conv; ++l) {
      const ConvSpec& C = Z.conv[l];
      const long long KK = C.K * C.K, HW = C.Hp * C.Wp;
      const std::string c = "conv" + std::to_string(l) + ".";
      t += "conv " + std::to_string(l);
      const std::pair<const char*, int> f[] = {
          {"Mi", C.Mi}, {"Hi", C.Hi}, {"Wi", C.Wi}, {"Mo", C.Mo}, {"Ho", C.Ho}, {"Wo", C.Wo}, {"K", C.K}, {"S", C.S},
          {"Kp", C.Kp}, {"Hp", C.Hp}, {"Wp", C.Wp}, {"max_conn", C.max_conn}, {"max_back", C.max_back},
          {"full_table", C.full_table}, {"n_own", C.n_own}, {"n_own_below", C.n_own_below},
          {"pull_shares", C.pull_shares}, {"back_pitch", C.back_pitch}, {"wgrad_R_log2", C.wgrad_R_log2},
          {"pull_chunk", C.pull_chunk}, {"fwd_strip", C.fwd_strip}, {"fwd_rows", C.fwd_rows},
          {"pull_strip", C.pull_strip}, {"pull_rows", C.pull_rows}, {"in_chunk", C.in_chunk}, {"pull_slots", C.pull_slots}};
      for (const auto& kv : f) t += std::string(" ") + kv.first + " " + std::to_string(kv.second);
      t += "\n";
      if (!(Z.stream && l >= 1)) region(c + "in", C.o_in, (long long)C.Mi * C.Hi * C.Wi);
      region(c + "wf", C.o_wf, (long long)C.n_own * C.max_conn * KK);
      region(c + "bf", C.o_bf, C.n_own);
      region(c + "cidx", C.o_cidx, (long long)C.n_own * C.max_conn);
      region(c + "ncf", C.o_ncf, C.n_own);
      if (l >= 1) {
        region(c + "wb", C.o_wb, (long long)C.n_own_below * C.back_pitch * KK);
        region(c + "bj", C.o_bj, (long long)C.n_own_below * C.back_pitch);
        region(c + "ncb", C.o_ncb, C.n_own_below);
        dall = std::max(dall, (long long)C.Mo * HW);
      }
      region(c + "pool", C.o_pool, C.n_own * HW);
      region(c + "yx", C.o_yx, C.n_own * HW);
      region(c + "delta", C.o_delta, C.n_own * HW);
      region(c + "dact", C.o_dact, C.n_own * HW);
      if (C.o_tab_fwd >= 0) region(c + "tab_fwd", C.o_tab_fwd, 3 * WG);
      if (C.o_tab_pull >= 0) region(c + "tab_pull", C.o_tab_pull, 3 * WG);
      act = std::max(act, (long long)C.n_own * C.Ho * C.Wo);
    }
    const ConvSpec& Cl = Z.conv[Z.n_conv - 1];
    for (int f = 0; f < Z.n_fc; ++f) {
      const FcSpec& Q = Z.fc[f];
      const std::string c = "fc" + std::to_string(f) + ".";
      t += "fc " + std::to_string(f) + " n_in " + std::to_string(Q.n_in) + " n_out " + std::to_string(Q.n_out) +
           " by_cols " + std::to_string(Q.by_cols) + " n_own " + std::to_string(Q.n_own) + "\n";
      region(c + "w", Q.o_w, f == 0 ? (long long)Cl.n_own * Cl.Hp * Cl.Wp * Q.n_out
                             : Q.by_cols ? (long long)Q.n_own * Q.n_out : (long long)Q.n_out * Q.n_in);
      region(c + "b", Q.o_b, Q.n_out);
      region(c + "act", Q.o_act, Q.n_out);
      region(c + "delta", Q.o_delta, Q.n_out);
      region(c + "dact", Q.o_dact, Q.n_out);
    }
    region("act", Z.o_act, act);
    // (the partial sums reach up to the next region: what they need is for the reader to work out)
    if (!Z.stream) region("part", Z.o_part, Z.o_dall - Z.o_part);
    if (Z.n_conv > 1) {
      region("dall", Z.o_dall, dall);
      region("yxall", Z.o_yxall, dall);
    }
    if (Z.defer && Z.n_conv > 1) region("prev", Z.o_prev, (long long)Z.conv[1].n_own_below * Z.conv[1].Hi * Z.conv[1].Wi);
    region("scratch", Z.o_scratch, Z.scratch_floats);
  }
  if (t.size() + 1 > n) return fail(nullptr, CNN_E_ARG, "buffer too small for the plan text");
  std::memcpy(buf, t.c_str(), t.size() + 1);
  return CNN_OK;
}

// development aid, host only: the plan of the batched forward pass of `arch` at `batch` images (tables as in
// cnn355_resident_plan_text), a line per trainable layer of "name value" pairs, then whether the output units
// add the planes of their layer's sums and the scratch floats a call takes (floats_32: with 32-bit products throughout, which
// is what a caller is asked for).
// split: the layer is a product of halves (k_batch_split), its tile, chunk and slab; first: the first layer below one (k_batch_first).  The values in front of these are then those of the product that the layer has without them.
// run: input maps (of KK terms each) of the longest running sum; gemm_run, gemm_KS: of k_batch_gemm's plan of the layer.
int cnn355_batch_plan_text(const char* arch, int fan_in, size_t batch, char* buf, size_t n) {
  if (!arch || !buf || n == 0 || batch == 0) return fail(nullptr, CNN_E_ARG, "NULL argument or batch of 0");
  cnn tmp;
  int rc = plan_only(tmp, arch, fan_in, 0, 0);
  if (rc) return rc;
  BatchPlan B;
  rc = batch_plan(&tmp, batch, B);
  if (rc) { g_err = tmp.err; return rc; }
  std::string t;
  for (const BatchStep& st : B.steps) {
    const BatchGemm& g = st.g;
    BatchConv c = st.c;
    std::vector<std::pair<const char*, long long>> f = {
        {"conv", c.MT != 0}, {"Mi", g.Mi}, {"KK", g.K * g.Kx}, {"gemm_KS", g.KS}, {"gemm_run", std::min(g.Mi, g.chunks_per_slice * g.IC)},
        {"wt_floats", (long long)st.wt_floats}};
    if (c.MT) {
      c.n_win = (int)(batch * c.win_img); c.n_cb = (c.n_win + c.wins - 1) / c.wins;
      f.insert(f.end(), {{"MT", c.MT}, {"TR", c.TR}, {"IC", c.IC}, {"n_slices", c.n_slices}, {"run", c.run}, {"resident", c.resident},
                         {"members", c.Kp * c.Kpx}, {"fuse", c.fuse}, {"wins", c.wins}, {"n_cb", c.n_cb}, {"gx", batch_conv_grid_x(c)},
                         {"groups", (c.Mo + c.MT * c.TR - 1) / (c.MT * c.TR)}, {"chunk_floats", c.IC * c.Hi * c.Wi},
                         {"lds_bytes", (long long)batch_conv_lds_bytes(c)}});
    } else {
      f.insert(f.end(), {{"MT", g.MT}, {"TR", g.TR}, {"IC", g.IC}, {"n_slices", g.KS},
                         {"run", std::min(g.Mi, g.chunks_per_slice * g.IC)}, {"members", g.Kp * g.Kpx}, {"fuse", g.fuse},
                         {"lds_bytes", (long long)batch_gemm_lds_bytes(g)}});
    }
    const BatchSplit& h = st.s;
    f.push_back({"split", h.RT != 0});
    f.push_back({"split_fc", h.fc && h.RT});
    f.push_back({"first", st.f.T != 0});
    if (st.f.T) f.insert(f.end(), {{"first_T", st.f.T}, {"first_H", st.f.H}, {"first_share", st.f.share}, {"first_shift", st.f.shift}, {"first_lds", (long long)batch_first_lds_bytes(st.f)}});
    if (h.RT)
      f.insert(f.end(), {{"split_RT", h.RT}, {"split_CT", h.CT}, {"split_TR", h.TR}, {"split_IC", h.IC}, {"split_kg", h.n_kg}, {"split_slab", h.slab},
                         {"split_slices", (h.n_cg / h.IC + h.cps - 1) / h.cps}, {"split_wins", h.wins}, {"split_px", h.run_px}, {"split_lds", (long long)batch_split_lds_bytes(h)}});
    t += "layer";
    for (const auto& kv : f) t += std::string(" ") + kv.first + " " + std::to_string(kv.second);
    t += "\n";
  }
  const BatchStep& last = B.steps.back();
  const bool add = last.raw() && outputs_add(tmp.prog.n_classes, last.pool.n_slices);
  t += "tail " + std::to_string((int)B.tail) + "\noutputs_add " + std::to_string((int)add) + "\nfloats " + std::to_string(B.floats(batch)) + "\nfloats_32 " + std::to_string(B.asked) + "\n";
  if (t.size() + 1 > n) return fail(nullptr, CNN_E_ARG, "buffer too small for the plan text");
  std::memcpy(buf, t.c_str(), t.size() + 1);
  return CNN_OK;
}

// development aid: how many ranks share the delta pull into one input map of the resident plan's conv layer l
int cnn355_resident_pull_shares(const cnn_t* net, int l) {
  if (!net || !net->flow_ok || l < 0 || l >= net->flow.n_conv) return -1;
  return net->flow.conv[l].pull_shares;
}

int cnn_set_team(cnn_t* net, int n_ranks, int xcd_stride) {
  if (!net || n_ranks < 0 || (xcd_stride != 0 && xcd_stride != 1 && xcd_stride != 8)) return CNN_E_ARG;
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  net->team_ranks = n_ranks;
  net->team_stride = xcd_stride;
  plan_flow(net);
  if (net->d_flow_ptrs)
    HIP_TRY(net, hipMemcpy(net->d_flow_ptrs, &net->flow_ptrs, sizeof(FlowPtrs), hipMemcpyHostToDevice));
  if (net->mode == CNN_MODE_RESIDENT && !net->flow_ok) {
    const std::string why = net->flow_why;
    const int rc = replan(net, CNN_MODE_PERSISTENT);
    return rc ? rc : fail(&net->err, CNN_E_STATE, why);
  }
  return CNN_OK;
}

int cnn_set_matrix_cores(cnn_t* net, int on) {
  if (!net) return CNN_E_ARG;
  if ((on != 0) == (net->use_mfma != 0)) return CNN_OK;
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  net->use_mfma = on ? 1 : 0;
  // re-plan the stages only: tables, weights and everything else on the device stay as they are
  int rc = plan(net);
  if (rc) return rc;
  HIP_TRY(net, hipMemcpy(net->d_prog, &net->prog, sizeof(ProgramDev), hipMemcpyHostToDevice));
  HIP_TRY(net, hipMemcpy(net->d_flow_ptrs, &net->flow_ptrs, sizeof(FlowPtrs), hipMemcpyHostToDevice));
  return CNN_OK;
}

int cnn_set_output_units(cnn_t* net, int kind) {
  if (!net || (kind != CNN_OUTPUT_SOFTMAX_XENT && kind != CNN_OUTPUT_TANH_SQERR)) return CNN_E_ARG;
  if (kind == net->out_units) return CNN_OK;
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  net->out_units = kind;
  // re-plan: the descriptors carry the kind; weights, tables and buffers stay as they are
  int rc = plan(net);
  if (rc) return rc;
  HIP_TRY(net, hipMemcpy(net->d_prog, &net->prog, sizeof(ProgramDev), hipMemcpyHostToDevice));
  HIP_TRY(net, hipMemcpy(net->d_flow_ptrs, &net->flow_ptrs, sizeof(FlowPtrs), hipMemcpyHostToDevice));
  return CNN_OK;
}

int cnn_get_output_units(const cnn_t* net) { return net ? net->out_units : CNN_E_ARG; }

int cnn_set_launch_graph(cnn_t* net, int images_per_graph) {
  if (!net || images_per_graph < 0 || images_per_graph > 1024) return fail(net ? &net->err : nullptr, CNN_E_ARG, "images_per_graph must lie in [0, 1024]");
  if (images_per_graph != net->graph_images) drop_stage_graphs(net);
  net->graph_images = images_per_graph;
  return CNN_OK;
}

int cnn_set_grid(cnn_t* net, int n_workgroups) {
  if (!net || n_workgroups < 0) return CNN_E_ARG;
  net->grid_override = n_workgroups;
  return CNN_OK;
}

int cnn_set_barrier(cnn_t* net, int kind) {
  if (!net || (kind != 0 && kind != 1)) return CNN_E_ARG;
  net->barrier_kind = kind;
  return CNN_OK;
}

int cnn_set_spin_limit(cnn_t* net, unsigned int polls) {
  if (!net) return CNN_E_ARG;
  net->spin_limit = polls;
  return CNN_OK;
}

int cnn_synchronize(cnn_t* net) {
  if (!net) return CNN_E_ARG;
  return sync_and_check(net);
}

int cnn_get_activation(cnn_t* net, int layer, float* host_dst) {
  if (!net || !host_dst) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (layer < 0 || layer >= (int)net->arch.size()) return fail(&net->err, CNN_E_ARG, "no such layer");
  int rc = sync_and_check(net);
  const ArchLayer& a = net->arch[layer];
  const size_t n = (size_t)a.maps * a.h * a.w;
  const float* src = nullptr;
  if (layer == 0) {
    if (!net->fe_n) return fail(&net->err, CNN_E_STATE, "layer 0 is the caller's image unless a front-end is set");
    src = net->d_fe_out;
  } else {
    const LayerDev& L = net->prog.layers[net->dev_of_arch[layer]];
    src = (a.kind == CNN_LAYER_POOL) ? L.out : L.act;
  }
  HIP_TRY(net, hipMemcpy(host_dst, src, n * sizeof(float), hipMemcpyDeviceToHost));
  return rc;
}

int cnn_get_delta(cnn_t* net, int layer, float* host_dst) {
  if (!net || !host_dst) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (layer < 1 || layer >= (int)net->arch.size() || net->arch[layer].kind == CNN_LAYER_POOL)
    return fail(&net->err, CNN_E_ARG, "deltas exist for convolutional and fully connected layers");
  int rc = sync_and_check(net);
  const ArchLayer& a = net->arch[layer];
  const LayerDev& L = net->prog.layers[net->dev_of_arch[layer]];
  if (a.kind == CNN_LAYER_FC) {
    HIP_TRY(net, hipMemcpy(host_dst, L.delta, (size_t)a.maps * sizeof(float), hipMemcpyDeviceToHost));
    return rc;
  }
  // scatter the winners' deltas back to the full-resolution map (index work only)
  const size_t small = (size_t)L.Mo * L.Hp * L.Wp, full = (size_t)L.Mo * L.Ho * L.Wo;
  std::vector<float> d(small);
  std::vector<int> yx(small);
  HIP_TRY(net, hipMemcpy(d.data(), L.delta, small * sizeof(float), hipMemcpyDeviceToHost));
  HIP_TRY(net, hipMemcpy(yx.data(), L.argyx, small * sizeof(int), hipMemcpyDeviceToHost));
  std::fill(host_dst, host_dst + full, 0.f);
  for (int j = 0; j < L.Mo; ++j)
    for (int q = 0; q < L.Hp * L.Wp; ++q) {
      const int v = yx[(size_t)j * L.Hp * L.Wp + q];
      const int y = v >> 16, x = v & 0xffff;
      if (y < 0 || y >= L.Ho || x >= L.Wo) continue;  // no forward pass has filled the winners yet
      host_dst[((size_t)j * L.Ho + y) * L.Wo + x] = d[(size_t)j * L.Hp * L.Wp + q];
    }
  return rc;
}

int cnn_get_argmax(cnn_t* net, int pool_layer, uint8_t* host_dst) {
  if (!net || !host_dst) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (pool_layer < 1 || pool_layer >= (int)net->arch.size() || net->arch[pool_layer].kind != CNN_LAYER_POOL)
    return fail(&net->err, CNN_E_ARG, "not a max-pooling layer");
  int rc = sync_and_check(net);
  const ArchLayer& a = net->arch[pool_layer];
  const LayerDev& L = net->prog.layers[net->dev_of_arch[pool_layer]];
  HIP_TRY(net, hipMemcpy(host_dst, L.arg, (size_t)a.maps * a.h * a.w, hipMemcpyDeviceToHost));
  return rc;
}

int cnn_get_loss(cnn_t* net, float* host_loss) {
  if (!net || !host_loss) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  StatusDev s;
  HIP_TRY(net, hipMemcpy(&s, net->d_status, sizeof(s), hipMemcpyDeviceToHost));
  *host_loss = s.loss;
  return check_status(net);
}

int cnn_get_stage_times(cnn_t* net, float* host_us, int max_stages, int* n_stages) {
  if (!net || !host_us || !n_stages) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  StatusDev s;
  HIP_TRY(net, hipMemcpy(&s, net->d_status, sizeof(s), hipMemcpyDeviceToHost));
  const int n = net->prog.n_stages;
  *n_stages = n;
  unsigned long long prev = s.stamps[0];
  for (int k = 0; k < n && k < max_stages; ++k) {
    const unsigned long long a = s.stamps[1 + 2 * k], b = s.stamps[2 + 2 * k];
    host_us[2 * k] = (a >= prev) ? (float)(a - prev) * 0.01f : 0.f;
    host_us[2 * k + 1] = (b >= a) ? (float)(b - a) * 0.01f : 0.f;
    if (b >= prev) prev = b;
  }
  return CNN_OK;
}

int cnn_debug_gradients(cnn_t* net, const float* d_image, int32_t label, float* host_grad) {
  if (!net || !d_image || !host_grad) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (label < 0 || label >= net->n_classes) return fail(&net->err, CNN_E_ARG, "label out of range");
  RunArgs a;
  std::memset(&a, 0, sizeof(a));
  a.images = d_image; a.n_images = 1; a.image_stride = (long long)net->image_size;
  a.label_imm = label; a.train = 1; a.lr = 0.f; a.grad_out = net->d_grad;
  int rc = run(net, a);
  if (rc) return rc;
  rc = sync_and_check(net);
  HIP_TRY(net, hipMemcpy(host_grad, net->d_grad, net->n_weights * sizeof(float), hipMemcpyDeviceToHost));
  return rc;
}

// development aid, not part of the public header: the raw device timestamps (100 MHz ticks) of the last call
int cnn355_read_status_stamps(cnn_t* net, unsigned long long* out, int n) {
  if (!net || !out) return CNN_E_ARG;
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  StatusDev s;
  HIP_TRY(net, hipMemcpy(&s, net->d_status, sizeof(s), hipMemcpyDeviceToHost));
  for (int i = 0; i < n && i < 2 * MAX_STAGES + 2; ++i) out[i] = s.stamps[i];
  return CNN_OK;
}

int cnn_measure_crossing(cnn_t* net, int n_ranks, int words_per_rank, int rounds, float* host_us) {
  if (!net || !host_us) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument");
  if (!net->coop_ok) return fail(&net->err, CNN_E_STATE, "device does not support cooperative launches");
  if (n_ranks < 2 || n_ranks > net->n_cu || words_per_rank < 1 || rounds < 1 || rounds > (1 << 20))
    return fail(&net->err, CNN_E_ARG, "cnn_measure_crossing: 2 to one rank per compute unit, at least one word and one round");
  if (2ull * n_ranks * words_per_rank > net->xbuf_words)
    return fail(&net->err, CNN_E_WORKSPACE, "cnn_measure_crossing: the network's exchange buffers hold " +
                std::to_string(net->xbuf_words / 2 / n_ranks) + " words per rank for this many ranks");
  const unsigned long long n = (unsigned long long)rounds + 1;
  HIP_TRY(net, hipStreamSynchronize(net->stream));
  if (((net->epoch + n) >> 32) != (net->epoch >> 32)) {
    net->epoch = ((net->epoch >> 32) + 1) << 32;
    HIP_TRY(net, hipMemset(net->d_xbuf, 0, net->xbuf_words * sizeof(tagged_t)));
  }
  HIP_TRY(net, launch_reset_status(net->stream, net->d_status, 0));
  const int stride = (n_ranks <= net->n_cu / 8) ? 8 : 1;
  HIP_TRY(net, launch_crossing_probe(n_ranks, stride, net->stream, net->d_xbuf, words_per_rank, rounds,
                                     (unsigned int)net->epoch, net->spin_limit, net->d_status));
  net->epoch += n;
  int rc = sync_and_check(net);
  if (rc) return rc;
  StatusDev s;
  HIP_TRY(net, hipMemcpy(&s, net->d_status, sizeof(s), hipMemcpyDeviceToHost));
  *host_us = (float)((double)(s.stamps[1] - s.stamps[0]) * 0.01 / rounds);
  return CNN_OK;
}

int cnn_measure_launch(cnn_t* net, int rounds, float* host_us) {
  if (!net || !host_us || rounds < 1) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument or no rounds");
  hipEvent_t e0, e1;
  HIP_TRY(net, hipEventCreate(&e0));
  HIP_TRY(net, hipEventCreate(&e1));
  for (int k = 0; k < 20; ++k) HIP_TRY(net, launch_empty(net->stream, net->d_status));
  HIP_TRY(net, hipEventRecord(e0, net->stream));
  for (int k = 0; k < rounds; ++k) HIP_TRY(net, launch_empty(net->stream, net->d_status));
  HIP_TRY(net, hipEventRecord(e1, net->stream));
  HIP_TRY(net, hipEventSynchronize(e1));
  float ms = 0.f;
  HIP_TRY(net, hipEventElapsedTime(&ms, e0, e1));
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *host_us = ms * 1e3f / (float)rounds;
  return CNN_OK;
}

// development aid, not part of the public header: in-item timestamps (zeros unless built with CNN355_STAMPS)
void cnn355_read_stamps(unsigned long long* out64) { cnn355::read_dbg(out64); }

const char* cnn_last_error(const cnn_t* net) { return net ? net->err.c_str() : g_err.c_str(); }

int cnn_forward_batch_scratch_bytes(cnn_t* net, size_t batch, size_t* bytes) {
  if (!net || !bytes || batch == 0) return fail(net ? &net->err : nullptr, CNN_E_ARG, "NULL argument or batch of 0");
  std::shared_ptr<const BatchKept> kept;
  int rc = batch_plan(net, batch, kept);
  if (rc) return rc;
  *bytes = kept->plan.asked * sizeof(float);
  return CNN_OK;
}

int cnn_deform_images(void* hip_stream, const float* d_src, size_t n_src, float* d_dst, size_t n, int C, int H, int W,
                      const cnn_deform_params* p, uint64_t seed, uint64_t first_index,
                      const int32_t* d_src_index, float* d_displacement) {
  if (n == 0) return CNN_OK;
  if (n_src == 0 || n_src > 0x7fffffffull || (!d_src_index && n > n_src))
    return fail(nullptr, CNN_E_ARG, "cnn_deform_images: more outputs than source images and no index list, or no source images");
  if (!d_src || !d_dst || !p) return fail(nullptr, CNN_E_ARG, "cnn_deform_images: NULL argument");
  if (d_src == d_dst) return fail(nullptr, CNN_E_ARG, "cnn_deform_images: source and destination must not overlap");
  if (C < 1 || H < 1 || W < 1 || (long long)H * (W | 1) > DEFORM_MAX_PIXELS || C > 1024)
    return fail(nullptr, CNN_E_SHAPE, "cnn_deform_images: rows x (columns rounded up to odd) at most 9312 (96 x 96), 1 to 1024 maps per image");
  if (n > (size_t)1 << 40) return fail(nullptr, CNN_E_ARG, "cnn_deform_images: too many images");
  const float ranges[6] = {p->max_translation, p->max_rotation, p->max_scaling, p->max_shear, p->sigma, p->fill};
  for (float r : ranges)
    if (!std::isfinite(r)) return fail(nullptr, CNN_E_ARG, "cnn_deform_images: a parameter is not finite");
  if (!std::isfinite(p->alpha)) return fail(nullptr, CNN_E_ARG, "cnn_deform_images: a parameter is not finite");
  if (p->max_translation < 0 || p->max_rotation < 0 || p->max_scaling < 0 || p->max_shear < 0 || p->sigma < 0)
    return fail(nullptr, CNN_E_ARG, "cnn_deform_images: a range or sigma is negative");
  if (p->max_scaling >= 1.0f) return fail(nullptr, CNN_E_ARG, "cnn_deform_images: max_scaling must be below 1");
  if (p->sigma > 16.0f) return fail(nullptr, CNN_E_ARG, "cnn_deform_images: sigma above 16 pixels");
  DeformJob J;
  J.src = d_src; J.dst = d_dst; J.disp = d_displacement; J.src_index = d_src_index;
  J.n = (long long)n; J.n_src = (long long)n_src; J.C = C; J.H = H; J.W = W;
  J.max_tx = (double)p->max_translation * W;
  J.max_ty = (double)p->max_translation * H;
  J.max_rot = (double)p->max_rotation / 180.0;
  J.max_shear = p->max_shear; J.max_scale = p->max_scaling; J.alpha = p->alpha; J.fill = p->fill;
  J.seed = seed; J.first_index = first_index;
  // |A - I| is at most 3 and 2 (1 + max_shear), the smoothed fields stay within [-1, 1]
  const double reach = 2.0 * (1.0 + J.max_shear) + 3.0;
  J.bounded = J.max_tx + J.max_ty + reach * (H + W) + std::fabs((double)J.alpha) < (double)(1 << 18);
  J.R = -1;
  for (float& t : J.taps) t = 0.f;
  if (p->sigma > 0.f && p->alpha != 0.f) {
    const double sg = p->sigma;
    const int R = (int)std::ceil(3.0 * sg);
    double g[2 * DEFORM_MAX_R + 1], sum = 0;
    for (int i = -R; i <= R; ++i) sum += g[i + R] = std::exp(-(double)i * i / (2.0 * sg * sg));
    for (int i = 0; i <= 2 * R; ++i) J.taps[i] = (float)(g[i] / sum);
    J.R = R;
  }
  hipError_t e = launch_deform((hipStream_t)hip_stream, J);
  if (e != hipSuccess) return fail(nullptr, CNN_E_HIP, std::string("cnn_deform_images: ") + hipGetErrorString(e));
  return CNN_OK;
}

// development aid, host only: 1 where the smoothing of such a call runs on the matrix cores, 0 where as sums over a line
int cnn355_deform_form(int C, int H, int W, float sigma) {
  DeformJob J;
  J.C = C; J.H = H; J.W = W; J.R = (int)std::ceil(3.0 * (double)sigma);
  return deform_mx_is_faster(J);
}

// tap_step >= 0 (parity tap): the pass stops behind that trainable layer and its outputs for the n <= batch
// images, [image][out_per_image], are copied to host_tap; d_probs is not written then.
static int forward_batch_impl(cnn_t* net, const float* d_images, size_t n, float* d_probs, void* d_scratch,
                              size_t scratch_bytes, size_t batch, int tap_step, float* host_tap, size_t* tap_per_image) {
  if (!net) return fail(nullptr, CNN_E_ARG, "NULL handle");
  if (n == 0) return CNN_OK;
  if (!d_images || (!d_probs && tap_step < 0) || !d_scratch || batch == 0) return fail(&net->err, CNN_E_ARG, "NULL argument or batch of 0");
  if (((uintptr_t)d_scratch & 255u) != 0) return fail(&net->err, CNN_E_ARG, "scratch must be 256-byte aligned");
  std::shared_ptr<const BatchKept> kept;
  int rc = batch_plan(net, batch, kept);
  if (rc) return rc;
  const BatchPlan& B = kept->plan;
  for (const BatchStep& st : B.steps) {
    const unsigned long long lim = (1ull << 31) - 256;
    const unsigned long long b = batch;
    if (b * (unsigned long long)st.g.P >= lim || b * (unsigned long long)st.g.out_stride >= lim ||
        b * (unsigned long long)st.g.in_stride >= lim || (unsigned long long)st.wt_floats >= lim)
      return fail(&net->err, CNN_E_ARG, "batch too large: the layer inputs and outputs of one batch must stay below 2^31 floats each");
  }
  if (net->prog.has_frontend && (unsigned long long)batch * net->image_size >= (1ull << 31) - 256)
    return fail(&net->err, CNN_E_ARG, "batch too large: the images of one batch must stay below 2^31 floats");
  if (scratch_bytes < B.floats(batch) * sizeof(float))
    return fail(&net->err, CNN_E_WORKSPACE, "scratch smaller than cnn_forward_batch_scratch_bytes says");
  if (tap_step >= 0 && (tap_step >= (int)B.steps.size() || n > batch || !host_tap))
    return fail(&net->err, CNN_E_ARG, "no such trainable layer, more images than one batch, or no buffer");
  const ProgramDev& P = net->prog;
  float* base = (float*)d_scratch;
  float* d_sums = base + B.wt_total;
  float* d_act[2] = {d_sums + batch * B.sums_per_image, d_sums + batch * (B.sums_per_image + B.act_per_image[0])};
  float* d_fe = d_act[1] + batch * B.act_per_image[1];
  // the weights as the products read them: one [k][map] matrix per layer, from their present values
  BatchPackAll pack;
  pack.n = (int)B.steps.size();
  for (int l = 0; l < pack.n; ++l) {
    pack.l[l] = B.steps[l].pack;
    pack.l[l].wt = base + B.steps[l].wt_off;
    const BatchSplit& h = B.steps[l].s;
    if (!h.RT) continue;
    const size_t rows = (size_t)(h.Mo + h.RT * h.TR - 1) / (h.RT * h.TR) * (h.RT * h.TR);
    pack.l[l].exps = (int*)(base + B.steps[l].wt_off + B.steps[l].wt_floats - up64(rows + 1));   // (behind the weights)
    pack.l[l].any = pack.l[l].exps + rows;
  }
  HIP_TRY(net, launch_batch_pack(net->stream, pack));
  const size_t fe_sz = P.has_frontend ? (size_t)P.fe.n_filters * P.fe.H * P.fe.W : 0;
  for (size_t t0 = 0; t0 < n; t0 += batch) {
    const size_t nb = std::min(batch, n - t0);
    const float* in = d_images + t0 * net->image_size;
    long long in_stride = (long long)net->image_size;
    if (P.has_frontend) {
      HIP_TRY(net, launch_frontend_batch(net->stream, net->d_prog, in, in_stride, (int)nb, (int)((fe_sz + WG - 1) / WG), d_fe));
      in = d_fe;
      in_stride = (long long)fe_sz;
    }
    int cur = 0;
    bool done = false;
    const BatchPool* last_raw = nullptr;
    SplitMarks in_marks = {nullptr, nullptr};
    for (size_t s = 0; s < B.steps.size(); ++s) {
      const BatchStep& st = B.steps[s];
      float* out = d_act[cur];
      const bool raw = st.raw();
      SplitMarks marks = {nullptr, nullptr};   // of the halves that this layer writes
      if (st.split_out) marks = {(unsigned char*)(out + batch * st.halves_per_image), pack.l[s + 1].any};
      if (st.f.T) {
        BatchFirst f = st.f;
        f.in = in; f.in_stride = in_stride; f.wt = base + st.wt_off; f.out = out; f.n_win = (int)(nb * f.win_img); f.out_marks = marks;
        HIP_TRY(net, launch_batch_first(net->stream, f));
      } else if (st.s.RT) {
        BatchSplit h = st.s;
        h.in = (const char*)in; h.wt = (const char*)(base + st.wt_off); h.exps = pack.l[s].exps; h.out = out;
        h.n_win = (int)(nb * h.win_img); h.n_cb = (h.n_win + h.wins - 1) / h.wins;
        h.in_marks = in_marks; h.out_marks = marks;
        if (h.raw) h.out = d_sums;
        HIP_TRY(net, launch_batch_split(net->stream, h));
      } else if (st.c.MT) {
        BatchConv c = st.c;
        c.in = in; c.in_stride = in_stride; c.wt = base + st.wt_off; c.out = raw ? d_sums : out;
        c.vec = ((uintptr_t)in & 15u) == 0 && in_stride % 4 == 0 && (c.IC * c.Hi * c.Wi) % 4 == 0 &&
                (c.n_slices == 1 || (c.run * c.Hi * c.Wi) % 4 == 0);
        c.n_win = (int)(nb * c.win_img); c.n_cb = (c.n_win + c.wins - 1) / c.wins;
        HIP_TRY(net, launch_batch_conv(net->stream, c));
      } else {
        BatchGemm g = st.g;
        g.in = in; g.in_stride = in_stride; g.wt = base + st.wt_off; g.N = (long long)nb * g.P; g.out = raw ? d_sums : out;
        HIP_TRY(net, launch_batch_gemm(net->stream, g));
      }
      if (raw && s + 1 == B.steps.size() && tap_step < 0 && outputs_add(P.n_classes, st.pool.n_slices)) {
        last_raw = &st.pool;
        in = d_sums;
        break;
      }
      const bool tail = B.tail && s + 2 == B.steps.size() && tap_step < 0;
      const bool add = tail && raw && st.pool.n_slices <= TAIL_SLICES;   // the planes are the last launch's too
      if (raw && !add) {
        BatchPool q = st.pool;
        q.sums = d_sums; q.out = out; q.total = (long long)nb * q.Mo * q.Hp * q.Wp;
        HIP_TRY(net, launch_batch_pool(net->stream, q));
      }
      if (tail) {
        const LayerDev& L = P.layers[P.n_layers - 1];
        BatchTail t;
        t.in = add ? d_sums : out; t.bias_h = add ? st.pool.bias : nullptr; t.w = L.w; t.bias = L.bias; t.out = d_probs + t0 * P.n_classes;
        t.n = (long long)nb; t.slice_stride = st.pool.slice_stride; t.n_slices = add ? st.pool.n_slices : 1;
        t.n_hidden = L.n_in; t.n_out = L.n_out; t.out_units = net->out_units; t.drop = B.steps.back().raw();
        HIP_TRY(net, launch_batch_tail(net->stream, t));
        done = true;
        break;
      }
      in = out;
      in_stride = (long long)st.out_per_image;
      in_marks = marks;
      cur ^= 1;
      if ((int)s == tap_step) {
        HIP_TRY(net, hipStreamSynchronize(net->stream));
        if (!st.split_out) {
          HIP_TRY(net, hipMemcpy(host_tap, out, nb * st.out_per_image * sizeof(float), hipMemcpyDeviceToHost));
          if (tap_per_image) *tap_per_image = st.out_per_image;
          return CNN_OK;
        }
        const size_t maps = (size_t)st.pool.Mo, pixels = (size_t)st.pool.Hp * st.pool.Wp;
        const BatchSplit& reader = B.steps[s + 1].s;
        const size_t eights = st.f.T ? st.f.T * 4 : st.s.RT * st.s.TR / 8;
        std::vector<unsigned short> halves(batch * st.halves_per_image * 2);
        std::vector<unsigned char> whole(reader.in_groups * batch * pixels);
        HIP_TRY(net, hipMemcpy(halves.data(), out, halves.size() * sizeof(halves[0]), hipMemcpyDeviceToHost));
        HIP_TRY(net, hipMemcpy(whole.data(), (const void*)marks.at, whole.size(), hipMemcpyDeviceToHost));
        for (size_t b = 0; b < nb; ++b)
          for (size_t j = 0; j < maps; ++j)
            for (size_t w = 0; w < pixels; ++w) {
              const unsigned short* h = &halves[((j >> 3) * 2 * batch * pixels + b * pixels + w) * 8 + (j & 7)];
              const unsigned short high = h[0], low = h[batch * pixels * 8];
              float& v = host_tap[(b * maps + j) * pixels + w];
              if (whole[(((j >> 3) + reader.in_shift) / eights * batch + b) * pixels + w]) v = __builtin_bit_cast(float, (unsigned)high << 16 | low);
              else v = ((float)__builtin_bit_cast(_Float16, high) + (float)__builtin_bit_cast(_Float16, low)) / (float)(1 << SPLIT_SHIFT);
            }
        if (tap_per_image) *tap_per_image = maps * pixels;
        return CNN_OK;
      }
    }
    if (done) continue;
    HIP_TRY(net, launch_batch_outputs(net->stream, in, last_raw ? last_raw->n_slices : 1, last_raw ? last_raw->slice_stride : 0,
                                      last_raw ? (const float*)last_raw->bias : nullptr, d_probs + t0 * P.n_classes, (long long)nb,
                                      P.n_classes, net->out_units));
  }
  return CNN_OK;
}

int cnn_forward_batch(cnn_t* net, const float* d_images, size_t n, float* d_probs, void* d_scratch,
                      size_t scratch_bytes, size_t batch) {
  return forward_batch_impl(net, d_images, n, d_probs, d_scratch, scratch_bytes, batch, -1, nullptr, nullptr);
}

int cnn_debug_forward_batch_layer(cnn_t* net, const float* d_images, size_t n, int trainable_layer, float* host_out,
                                  size_t* host_floats_per_image, void* d_scratch, size_t scratch_bytes) {
  return forward_batch_impl(net, d_images, n, nullptr, d_scratch, scratch_bytes, n, trainable_layer, host_out,
                            host_floats_per_image);
}

}  // extern "C"

// ---- the batched forward pass for callers that cannot allocate ------------------------------------
// cnn_forward_batch takes its scratch memory from the caller.  This variant takes it from an array that
// is part of the library's device image instead, so that the call allocates nothing anywhere.  In host
// code the array's name only stands for the symbol: the address of the memory on the device that is
// current comes from hipGetSymbolAddress, once per device (every device holds its own copy), and only
// that address is ever used.
namespace {
constexpr size_t STATIC_SCRATCH_BYTES = (size_t)CNN_FORWARD_BATCH_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];
constexpr int STATIC_SCRATCH_MAX_DEVICES = 64;
void* g_scratch_ptr[STATIC_SCRATCH_MAX_DEVICES] = {};
std::mutex g_scratch_mutex;

// the array's address on the current device (asked for once per device), or NULL with *err set
void* static_scratch_ptr(hipError_t* err, int* device) {
  *err = hipGetDevice(device);
  if (*err != hipSuccess) return nullptr;
  if (*device < 0 || *device >= STATIC_SCRATCH_MAX_DEVICES) { *err = hipErrorInvalidDevice; return nullptr; }
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[*device]) {
    void* p = nullptr;
    *err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (*err != hipSuccess || !p) { if (*err == hipSuccess) *err = hipErrorInvalidSymbol; return nullptr; }
    g_scratch_ptr[*device] = p;
  }
  return g_scratch_ptr[*device];
}
}  // namespace

extern "C" int cnn_forward_batch_static(cnn_t* net, const float* d_images, size_t n, float* d_probs, size_t batch) {
  if (!net) return fail(nullptr, CNN_E_ARG, "NULL handle");
  if (n == 0) return CNN_OK;
  if (!d_images || !d_probs || batch == 0) return fail(&net->err, CNN_E_ARG, "NULL argument or batch of 0");
  size_t need = 0;
  int rc = cnn_forward_batch_scratch_bytes(net, batch, &need);
  if (rc) return rc;
  if (need > STATIC_SCRATCH_BYTES)
    return fail(&net->err, CNN_E_WORKSPACE, "cnn_forward_batch_static: a batch of " + std::to_string(batch) + " images needs " +
                std::to_string(need) + " bytes of scratch, the library's own array holds " +
                std::to_string(STATIC_SCRATCH_BYTES) + ": use a smaller batch, or cnn_forward_batch with memory of the caller's");
  hipError_t e = hipSuccess;
  int device = -1;
  void* ptr = static_scratch_ptr(&e, &device);
  if (!ptr) return hip_fail(net, e, "cnn_forward_batch_static: address of the scratch array");
  if (device != net->device)
    return fail(&net->err, CNN_E_STATE, "cnn_forward_batch_static: the current device is not the one the network was created on");
  return cnn_forward_batch(net, d_images, n, d_probs, ptr, STATIC_SCRATCH_BYTES, batch);
}
