// The layer's host code (csrc/dgc_api.hip holds no kernel) on stand-ins of the HIP runtime and of the kernels' launchers:
// device memory is host memory, the n-th allocation can be made to fail, launches leave their names and their pointers in
// a log.  Called by test_host_layer.py with the name of a check; a check that fails says so and ends the program with 1.
#include "dgc_api.hip"

#include <cstdio>
#include <cstdlib>

static std::vector<std::string> calls;      // launches and stream operations, in order
static int allocations = 0, fails_at = 0;   // the fails_at-th allocation fails (0: none)
static size_t bytes_allocated = 0;          // of device memory
static hipError_t last_error = hipSuccess;
static int device = 0;
static bool null_pointer = false;           // a launcher was handed one

static void launched(const char* name, std::initializer_list<const void*> pointers) {
  calls.push_back(name);
  for (const void* p : pointers) null_pointer |= p == nullptr;
}
static int count(const char* name) { return (int)std::count(calls.begin(), calls.end(), name); }
static void expect(bool ok, const char* what) {
  if (ok) return;
  std::printf("not so: %s\n", what);
  std::exit(1);
}

static std::string fails;                   // the call of this name fails
static hipError_t next_call(const std::string& name) {
  calls.push_back(name);
  return name == fails ? last_error = hipErrorUnknown : hipSuccess;
}

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  bytes_allocated += n;
  if (++allocations == fails_at) return last_error = hipErrorOutOfMemory;
  *p = std::calloc(n ? n : 1, 1);
  return hipSuccess;
}
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last_error; last_error = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "out of memory"; }
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(to, from, n); return hipSuccess; }
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind) { std::memcpy(to, from, n); return next_call("copy"); }
hipError_t hipMemset(void* p, int value, size_t n) { std::memset(p, value, n); return next_call("clear"); }
hipError_t hipDeviceSynchronize() { return next_call("wait for the device"); }
static float* finished_by_waiting = nullptr;      // a number that the device still writes: there after the default stream has been waited for
hipError_t hipStreamSynchronize(hipStream_t s) {
  const hipError_t e = next_call("wait for stream " + std::to_string(reinterpret_cast<uintptr_t>(s)) + " of device " + std::to_string(device));
  if (e == hipSuccess && finished_by_waiting) *finished_by_waiting += 1.f;
  return e;
}
hipError_t hipSetDevice(int d) { device = d; return next_call("device " + std::to_string(d)); }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { calls.push_back("wait"); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  calls.push_back("event " + std::to_string(reinterpret_cast<uintptr_t>(e)));
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
  *ms = (float)(reinterpret_cast<uintptr_t>(b) - reinterpret_cast<uintptr_t>(a));
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int bytes) {
  calls.push_back("allow " + std::to_string(bytes));
  return fails_at < 0 ? hipErrorInvalidValue : hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(n, 1); return hipSuccess; }
hipError_t hipMemsetAsync(void* p, int value, size_t n, hipStream_t) { std::memset(p, value, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
}

namespace dgc {
void launch_spmm(const SpmmArgs& a, hipStream_t) { launched("spmm", {a.fresh, a.M}); if (a.skip_stale) null_pointer |= !a.row_map; }
bool launch_dense(const DenseArgs& a, hipStream_t, std::string*) {
  launched(a.Wf ? "folded dense" : "dense", {a.M, a.Wg, a.Y});
  if (a.Wf) null_pointer |= !a.bf || !a.fold_bad;
  return true;
}
void launch_fold(const float* wih, int64_t, const float* wg, const float* bg, const float* bih, int32_t, int32_t, int32_t, float* out, float* bias,
                 int32_t* bad, hipStream_t) {
  launched("fold", {wih, wg, bg, bih, out, bias, bad});
}
void launch_pack_split(const float* w, int64_t, int64_t, int64_t, int32_t, int32_t, int64_t, void* packed, hipStream_t) {
  launched("pack weight", {w, packed});
}
void launch_inside(const SpmmArgs& a, int64_t* eptr, int2* inside, hipStream_t) {
  launched(inside ? "fill neighbours" : "count neighbours", {a.etab, eptr});
}
void launch_exclusive_scan(int64_t* data, int64_t, int64_t* tmp, int64_t* total, hipStream_t) { launched("scan", {data, tmp, total}); }
int64_t scan_tmp_elems(int64_t) { return 4; }
void launch_edge_table(const GraphDev&, const Segment*, int64_t, int64_t, const float*, const int32_t*, int2* etab, hipStream_t) {
  launched("edge table", {etab});
}
bool dense_narrow_wanted(int32_t, int32_t, bool, int64_t, int32_t) { return false; }
void evolve_forward_weights(const EvolveWs&, hipStream_t) { launched("recurrence", {}); }
bool evolve_backward_dw(const EvolveWs&, const EvolveBwdIn&, bool, hipStream_t, std::string*) { launched("weight gradient", {}); return true; }
void evolve_backward_bptt(const EvolveWs&, hipStream_t) { launched("back-propagation", {}); }
int32_t evolve_dw_split(int32_t, int32_t, int64_t most_tiles) { return (int32_t)std::min<int64_t>(8, most_tiles); }
int64_t evolve_partial_elems(const EvolveWs& ws) { return (int64_t)ws.T * ws.split_dw * ws.F * ws.S; }
int64_t evolve_loss_partial_elems(const EvolveWs& ws) { return (int64_t)ws.T * ws.split_dw; }
bool dense_split_supported(int32_t, int32_t, int32_t) { return true; }
void evolve_row_index(const ChunkInfo*, int32_t, int64_t, int32_t, int64_t, int64_t* idx, hipStream_t) { launched("row index", {idx}); }
void evolve_pack_weights_plain(const EvolveWs&, float4* packed, hipStream_t) { launched("pack", {packed}); }
void labels_build(const GraphDev&, const Segment*, const int32_t*, int32_t* col, int64_t* in, int64_t* out, hipStream_t) {
  launched("labels", {col, in, out});
}
}  // namespace dgc

// An EvolveGCN-O layer of one chunk, 2 snapshots x 40 vertices, width 32, after its forward.
static dgc_layer* evolve_layer() {
  static float memory[64];
  static int64_t index[3] = {0, 2, 4};
  dgc_layer* L = new dgc_layer();
  L->desc.struct_kind = DGC_STRUCT_EVOLVE_GCN_O;
  L->desc.n_struct_layers = 1;
  L->desc.F = L->desc.S = L->desc.H = 32;
  L->desc.act_out = DGC_ACT_RELU;
  L->T = 2; L->N = 40; L->n_chunks = 1;
  L->chunks = {dgc_chunk_t{0, 40, 0, 2}};
  L->total_rows = 80; L->total_nnz = 80;
  L->cinfo_host = {ChunkInfo{0, 40, 0, 0, 0, 2}};
  L->row_tile_ptr.assign(index, index + 3);
  L->evo.T = 2; L->evo.F = L->evo.S = 32; L->evo.split = true;
  L->d_M = memory; L->ldm = 32;
  L->evo.Wt_packed = reinterpret_cast<float4*>(memory);
  L->side = reinterpret_cast<hipStream_t>(uintptr_t(1));
  L->fork = reinterpret_cast<hipEvent_t>(uintptr_t(101));
  L->join = reinterpret_cast<hipEvent_t>(uintptr_t(102));
  L->forward_done = L->m_saved = true;
  return L;
}
alignas(16) static float tensor[64];

// Whichever buffer of the input gradient there is no memory for: the call reports it and starts nothing of the input
// gradient, and so does the next call; the parameters' gradients are computed; with memory the next call does it all.
static void input_gradient_memory() {
  for (int n = 1; n <= 3; ++n) {
    dgc_layer* L = evolve_layer();
    auto backward = [&] { return dgc_layer_backward(L, tensor, 32, nullptr, 0, tensor, 32, nullptr, tensor, 32, nullptr); };
    calls.clear();
    for (int attempt = 0; attempt < 2; ++attempt) {
      allocations = 0; fails_at = n;
      expect(backward() != DGC_OK, "a backward without memory for the input gradient is an error");
      expect(allocations == n, "the buffers are asked for one after the other");
      expect(count("weight gradient") == attempt + 1 && count("back-propagation") == attempt + 1, "the parameters' gradients are computed");
      expect(count("row index") + count("pack") + count("dense") + count("spmm") == 0, "nothing of the input gradient is started");
      expect(L->allocs.empty(), "what was allocated is given back");
      expect(hipGetLastError() == hipSuccess, "no error is left for a later call");
    }
    fails_at = 0;
    expect(backward() == DGC_OK, "with memory it works");
    expect(count("row index") == 1 && count("pack") == 1 && count("dense") == 1 && count("spmm") == 1 && !null_pointer,
           "the input gradient is computed from buffers that are there");
    L->m_saved = true;
    expect(backward() == DGC_OK && count("row index") == 1 && L->allocs.size() == 3, "the buffers are kept");
  }
}

static void label_memory() {
  for (int n = 1; n <= 4; ++n) {
    dgc_layer* L = evolve_layer();
    std::vector<int32_t> labels(80, 0);
    calls.clear();
    for (int attempt = 0; attempt < 2; ++attempt) {
      allocations = 0; fails_at = n;
      expect(dgc_layer_set_labels(L, labels.data(), nullptr) != DGC_OK, "labels without memory are an error");
      expect(calls.empty() && L->allocs.empty() && !L->lab.built, "nothing is started or kept");
    }
    fails_at = 0;
    expect(dgc_layer_set_labels(L, labels.data(), nullptr) == DGC_OK && count("labels") == 1 && !null_pointer, "with memory it works");
  }
}

// The input gradient's table of neighbours: without memory for it the gradient is computed without it; a labelled layer's keeps its place
// and is filled by every set_labels from the first dX on, and only there.
static void neighbour_table() {
  static int2 etab[128];
  static int64_t begins[96];
  for (int n = 0; n <= 1; ++n) {             // two chunks with neighbours in each other
    dgc_layer* L = evolve_layer();
    L->chunks = {dgc_chunk_t{0, 20, 0, 2}, dgc_chunk_t{20, 40, 0, 2}};
    L->n_chunks = 2;
    L->d_etab = etab; L->d_inside_ptr = begins; L->n_inside = 60;
    calls.clear();
    allocations = 0; fails_at = n;
    expect(dgc_layer_backward(L, tensor, 32, nullptr, 0, tensor, 32, nullptr, tensor, 32, nullptr) == DGC_OK, "the input gradient is computed");
    expect(count("fill neighbours") == 1 - n && (L->d_inside != nullptr) == (n == 0) && count("spmm") == 1 && !null_pointer, "with the table if there is memory for it");
    expect(hipGetLastError() == hipSuccess, "no error is left for a later call");
    L->m_saved = true;
    allocations = 0;
    expect(dgc_layer_backward(L, tensor, 32, nullptr, 0, tensor, 32, nullptr, tensor, 32, nullptr) == DGC_OK && allocations == 0 &&
           count("fill neighbours") == 1 - n, "the next one as well");
  }
  fails_at = 0;
  dgc_layer* L = evolve_layer();
  L->d_etab = etab;
  std::vector<int32_t> labels(80, 0);
  auto backward = [&] { L->forward_done = L->m_saved = true; return dgc_layer_backward(L, tensor, 32, nullptr, 0, tensor, 32, nullptr, tensor, 32, nullptr); };
  calls.clear();
  expect(dgc_layer_set_labels(L, labels.data(), nullptr) == DGC_OK && count("fill neighbours") == 0, "no table before the first dX");
  expect(backward() == DGC_OK && count("fill neighbours") == 1, "the first dX makes it");
  const int2* const place = L->d_inside;
  allocations = 0;
  expect(dgc_layer_set_labels(L, labels.data(), nullptr) == DGC_OK && count("fill neighbours") == 2 && allocations == 0 && L->d_inside == place,
         "other labels fill it where it is");
  expect(backward() == DGC_OK && count("fill neighbours") == 2 && allocations == 0, "a backward does not");
  L = evolve_layer();
  L->d_etab = etab;
  calls.clear();
  expect(backward() == DGC_OK && !L->d_inside && count("fill neighbours") == 0, "no table without labels");
  allocations = 0; fails_at = 5;             // (the labels take four)
  expect(dgc_layer_set_labels(L, labels.data(), nullptr) == DGC_OK && !L->d_inside && L->lab.built, "labels need no table");
  expect(backward() == DGC_OK && count("spmm") == 2, "nor does the gradient");
  fails_at = 0;
  expect(dgc_layer_set_labels(L, labels.data(), nullptr) == DGC_OK && L->d_inside && count("fill neighbours") == 1 && !null_pointer, "later ones make it");
}

// What an EvolveGCN-O layer keeps per snapshot beside the partial sums of the weight gradients: the weights and gates in double,
// the weights in fp32 and packed, their direct gradient.  The gradients of the gates' arguments are not on top of that.
static void evolve_memory() {
  for (int64_t tiles : {8, 3}) {
    dgc_layer L;
    L.desc.struct_kind = DGC_STRUCT_EVOLVE_GCN_O;
    L.desc.F = L.desc.S = 64;
    L.T = 200;
    for (int64_t t = 0; t <= L.T; ++t) L.row_tile_ptr.push_back(t * tiles);
    bytes_allocated = 0;
    expect(build_evolve(&L, {}, nullptr) == DGC_OK, "the layer is built");
    const size_t n = 64 * 64, per_snapshot = n * (4 * sizeof(double) + sizeof(float) + 6 + sizeof(float));
    const size_t partial = n * sizeof(float) * std::max<size_t>(tiles, 6), once = n * 48 * sizeof(float) + 65536;
    expect(bytes_allocated <= 200 * (per_snapshot + partial) + once, "memory is that of the partial sums, the weights and the gates");
    const char *first = reinterpret_cast<char*>(L.evo.partial), *end = first + 200 * partial;
    for (double* a : {L.evo.Ah, L.evo.Az, L.evo.Ar})
      expect(reinterpret_cast<char*>(a) >= first && reinterpret_cast<char*>(a + 200 * n) <= end, "the arguments' gradients lie in it");
  }
}

// The events around a stage enclose its launches and nothing else: the caller's stream waits for the weight recurrence
// after the aggregation's last event and before the dense stage's first; no stage 1 or 2 without a second GCN layer.
static void stage_events() {
  dgc_layer* L = evolve_layer();
  for (int i = 0; i <= DGC_N_STAGES; ++i) L->ev[i] = reinterpret_cast<hipEvent_t>(uintptr_t(1 + 10 * i));
  for (int i = 0; i < 6; ++i) L->evx[i] = reinterpret_cast<hipEvent_t>(uintptr_t(1001 + 10 * i));
  L->profiling = true;
  calls.clear();
  expect(dgc_layer_forward(L, tensor, 32, tensor, 32, nullptr, 0, nullptr, nullptr, tensor, 32, nullptr, nullptr) == DGC_OK, "forward");
  auto at = [&](const char* name, int nth = 0) {
    for (size_t i = 0; i < calls.size(); ++i)
      if (calls[i] == name && nth-- == 0) return (int)i;
    return -1;
  };
  expect(count("wait") == 2 && at("wait", 0) < at("recurrence"), "the recurrence's stream waits for the caller's, then the caller's for it");
  const int join = at("wait", 1);
  expect(at("event 1") >= 0 && at("event 1") < at("spmm") && at("event 11") == at("spmm") + 1, "stage 0 is the aggregation");
  expect(at("event 11") < join && join < at("event 31"), "no stage holds the wait");
  expect(at("event 31") == at("dense") - 1 && at("event 41") == at("dense") + 1, "stage 3 is the dense kernel");
  expect(at("event 1001") == at("recurrence") - 1 && at("event 1011") == at("recurrence") + 1, "stage 4 is the recurrence");
  float ms[DGC_N_STAGES];
  expect(dgc_layer_stage_times(L, ms) == DGC_OK, "stage times");
  expect(ms[0] == 10 && ms[1] == 0 && ms[2] == 0 && ms[3] == 10 && ms[4] == 10 && ms[5] == 0, "the stages that ran");
  calls.clear();
  expect(dgc_layer_backward(L, tensor, 32, nullptr, 0, tensor, 32, nullptr, tensor, 32, nullptr) == DGC_OK, "backward");
  expect(at("event 1021") == at("weight gradient") - 1 && at("event 1031") == at("weight gradient") + 1, "stage 5 is the weight gradient");
  expect(at("event 1041") == at("back-propagation") - 1 && at("event 1051") == at("back-propagation") + 1, "stage 6 is the back-propagation");
  expect(calls.back() == "wait", "the caller's stream waits for the other one");
}

// A gradient is read after the default stream of the layer's device has been waited for, whichever device is current, and not
// at all if the wait fails; the caller's device is current again in either case.
static void gradient_read() {
  dgc_layer L;
  float there[2] = {1.f, 2.f}, out[2];
  Param p;
  p.raw = there; p.on_host = true; p.n_out = 2;
  L.params["x.grad"] = p;
  L.device = 1;
  finished_by_waiting = there + 1;
  for (int current : {0, 1}) {
    device = current;
    calls.clear();
    out[0] = out[1] = -1.f;
    there[1] = 2.f;
    expect(dgc_layer_get_param(&L, "x.grad", out, 2) == DGC_OK && out[0] == 1.f && out[1] == 3.f, "what is read has been finished");
    expect(device == current && count("wait for stream 0 of device 1") == 1 && count("copy") == 0, "the layer's device is waited for");
    expect((int)calls.size() == (current == 1 ? 1 : 3), "and made current only where it is not");
    fails = "wait for stream 0 of device 1";
    out[0] = -1.f;
    expect(dgc_layer_get_param(&L, "x.grad", out, 2) == DGC_ERR_DEVICE && out[0] == -1.f && device == current, "a failed wait is reported");
    fails.clear();
  }
  expect(dgc_layer_get_param(&L, "x.grad", out, 3) == DGC_ERR_INVALID_ARG && dgc_layer_set_param(&L, "x.grad", out, 2) == DGC_ERR_INVALID_ARG,
         "sizes are checked, gradients are not set");
  finished_by_waiting = nullptr;
}

// The folded weights are made when the last of the four parameters has been set, and again whenever one of them is; a forward
// takes them only if the last attempt succeeded.
static void folded_weights() {
  dgc_layer* L = new dgc_layer();
  L->desc.struct_kind = DGC_STRUCT_GCN;
  L->desc.time_kind = DGC_TIME_GRU;
  L->desc.n_struct_layers = 1;
  L->desc.F = L->desc.S = L->desc.H = 32;
  L->T = 2; L->N = 40; L->n_chunks = 1;
  L->d_M = tensor; L->ldm = 32;
  std::vector<float> v(96 * 32, 0.5f);
  const std::vector<std::string> names = {"gcn0.weight", "gcn0.bias", "rnn.weight_ih", "rnn.weight_hh", "rnn.bias_ih", "rnn.bias_hh"};
  for (const std::string& name : names) {
    const bool rnn = name[0] == 'r', weight = name.find("weight") != std::string::npos;
    expect(add_param(L, name, rnn ? 96 : 32, weight ? 32 : 0, nullptr, true) == DGC_OK, "a parameter");
  }
  L->fold.may = true;
  expect(dev_alloc_all(L, Wanted<float>{&L->fold.W, 96 * 32}, Wanted<float>{&L->fold.bias, 96}, Wanted<float4>{&L->fold.packed, 96 * 32},
                       Wanted<int32_t>{&L->fold.bad, 1}) == hipSuccess, "memory");
  auto set = [&](const std::string& name) { return dgc_layer_set_param(L, name.c_str(), v.data(), L->params[name].numel()); };
  auto folds = [&] {
    calls.clear();
    expect(dgc_layer_forward(L, tensor, 32, tensor, 32, nullptr, 0, nullptr, nullptr, tensor, 32, nullptr, nullptr) == DGC_OK, "forward");
    expect(count("folded dense") + count("dense") == 1 && !null_pointer, "one time encoder, on weights that are there");
    return count("folded dense") == 1;
  };
  for (size_t k = 0; k < names.size(); ++k) {
    calls.clear();
    expect(set(names[k]) == DGC_OK && count("fold") == (k == 4), "made with the last of the four");
    expect(folds() == (k >= 4), "and used from then on");
  }
  for (const char* where : {"clear", "wait for the device"}) {
    fails = where;
    expect(set("gcn0.bias") == DGC_ERR_DEVICE && hipGetLastError() != hipSuccess && !folds(), "after an error the transform runs");
    fails.clear();
    calls.clear();
    expect(set("rnn.bias_ih") == DGC_OK && count("fold") == 1 && folds(), "until the next parameter");
  }
}

// One or two snapshots of streamed matrices evolve on the caller's stream, before the aggregation and the transform.
static void one_stream() {
  for (int T : {1, 2, 3}) {
    dgc_layer* L = evolve_layer();
    L->T = T;
    L->desc.F = L->desc.S = L->desc.H = 96;
    calls.clear();
    expect(dgc_layer_forward(L, tensor, 96, tensor, 96, nullptr, 0, nullptr, nullptr, tensor, 96, nullptr, nullptr) == DGC_OK, "forward");
    expect(count("recurrence") == 1 && count("spmm") == 1 && count("dense") == 1, "its launches");
    if (T <= 2) expect(calls == std::vector<std::string>({"recurrence", "spmm", "dense"}), "no event, in this order");
    else expect(count("wait") == 2, "more snapshots: beside the aggregation");
  }
}

// Large dynamic LDS is allowed once on every device that a kernel runs on; a refusal is reported and not taken for done.
static void lds_per_device() {
  std::atomic<uint64_t> done{0};
  std::string why;
  calls.clear();
  for (int pass = 0; pass < 2; ++pass)
    for (device = 0; device < 3; ++device) expect(allow_lds(&done, 98304, done, &why), "it is allowed");
  expect(count("allow 98304") == 3, "once on each device");
  fails_at = -1;
  device = 5;
  expect(!allow_lds(&done, 98304, done, &why) && !why.empty(), "a refusal is reported");
  fails_at = 0;
  expect(allow_lds(&done, 98304, done, &why) && count("allow 98304") == 5, "and asked for again");
}

int main(int argc, char** argv) {
  const std::string check = argc > 1 ? argv[1] : "";
  if (check == "input gradient memory") input_gradient_memory();
  else if (check == "label memory") label_memory();
  else if (check == "neighbour table") neighbour_table();
  else if (check == "stage events") stage_events();
  else if (check == "lds per device") lds_per_device();
  else if (check == "one stream") one_stream();
  else if (check == "evolve memory") evolve_memory();
  else if (check == "gradient read") gradient_read();
  else if (check == "folded weights") folded_weights();
  else expect(false, "the check is known");
  std::puts("so");
  return 0;
}
