// Host-side check of what scratch memory the library asks for and how it does with
// less, and of calls under stream capture with saved tile choices
// (tests/test_scratch_host.py).  The HIP runtime's calls are answered here: device
// memory is numbers from a counter, an allocation past `device_free` fails, a wait
// fails while `capturing`, launches and copies do nothing.  So whole entry points run on a machine without a GPU.
#include <stdio.h>
#include <string.h>

#include <algorithm>

#include "rif_internal.hpp"

static size_t device_free = ~size_t(0);   // largest single allocation that succeeds
static size_t n_malloc = 0, n_denied = 0, n_launch = 0, n_coop = 0;
static bool capturing = false;
extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  static size_t next = 1 << 20;
  ++n_malloc;
  if (n > device_free) { ++n_denied; *p = nullptr; return hipErrorOutOfMemory; }
  *p = (void*)next;
  next += (n + 4095) & ~size_t(4095);
  return hipSuccess;
}
hipError_t hipFree(void*) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { ++n_launch; return hipSuccess; }
hipError_t hipLaunchCooperativeKernel(const void*, dim3, dim3, void**, unsigned, hipStream_t) { ++n_coop; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return capturing ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return capturing ? hipErrorStreamCaptureUnsupported : hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)16; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)16; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = (hipEvent_t)16; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 1;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return hipSuccess; }
}

static int n_fail = 0, n_check = 0;
static void check(bool ok, const char* what, size_t a = 0, size_t b = 0) {
  ++n_check;
  if (ok) return;
  ++n_fail;
  printf("FAIL %s (%zu, %zu)\n", what, a, b);
}

static double word;   // every operand's "address"
static rif_instance molecule(int nb, int na, int npairs, int ncwo, int nmo) {
  rif_instance in;
  memset(&in, 0, sizeof in);
  double* p = &word;
  in.n_bf = nb; in.n_aux = na; in.n_pairs = npairs; in.n_cwo = ncwo; in.n_mo = nmo;
  in.b = in.C = in.H = in.occ = p;
  in.b_half = in.b_mo = in.Jn = in.Kn = p;
  in.d = in.J = in.K = in.energy = in.lambda = in.grad = p;
  return in;
}

// What `call` asks for without a limit, and the smallest limit it runs with.
template <class Call>
static size_t free_size(Call&& call) {
  rif_ctx c;
  check(call(&c) == RIF_OK, "call without a limit");
  return c.ws_bytes;
}
template <class Call>
static bool runs_with(size_t limit, Call&& call) {
  rif_ctx c;
  c.ws_limit = limit;
  const bool ok = call(&c) == RIF_OK;
  check(c.ws_bytes <= std::max(limit, (size_t)1 << 20), "arena past the limit", c.ws_bytes, limit);
  return ok;
}
template <class Call>
static size_t least_size(Call&& call) {
  size_t lo = 0, hi = free_size(call);
  while (hi - lo > 1) {
    const size_t mid = lo + (hi - lo) / 2;
    (runs_with(mid, call) ? hi : lo) = mid;
  }
  return hi;
}
// With a device that has the least but not all: the call runs, runs again without
// another allocation, and takes all once it is there and the limit is set anew.
template <class Call>
static void on_a_full_device(const char* what, Call&& call) {
  const size_t full = free_size(call), least = std::max(least_size(call), (size_t)1 << 20);
  rif_ctx c;
  device_free = least;
  check(call(&c) == RIF_OK && c.err.empty(), what, least, full);
  check(c.ws_bytes == least, what, c.ws_bytes, least);
  const size_t before = n_malloc;
  check(call(&c) == RIF_OK && n_malloc == before, what, n_malloc, before);
  device_free = ~size_t(0);
  rif_set_workspace_limit(&c, 0);
  check(call(&c) == RIF_OK && c.ws_bytes == full, what, c.ws_bytes, full);
  device_free = least - 1;
  rif_ctx d;
  check(call(&d) == RIF_ENOMEM, what, least, full);
  device_free = ~size_t(0);
}

static void builds() {
  const rif_instance in = molecule(400, 8, 100, 3, 400);
  auto build = [&](rif_prec prec) { return [&in, prec](rif_ctx* c) { return rif_build(c, &in, prec, RIF_PNOF7); }; };
  auto energy = [&](rif_prec prec) {
    return [&in, prec](rif_ctx* c) {
      return pnof_energy_grad(c, RIF_PNOF7, 400, 400, 100, 3, nullptr, &word, &word, &word, &word, &word, &word, &word,
                              prec, &word, &word, &word);
    };
  };
  const rif_prec modes[] = {RIF_FP32, RIF_BF16X3, RIF_BF16X6, RIF_FP16X3};
  // FP64 works in more than it needs (the Fock step's strips); the other modes have no use for more
  check(least_size(build(RIF_FP64)) < free_size(build(RIF_FP64)), "FP64 build: strips' partials");
  for (rif_prec p : modes) {
    check(free_size(build(p)) == least_size(build(p)), "build holds what it does not use", free_size(build(p)), least_size(build(p)));
    check(free_size(energy(p)) == least_size(energy(p)), "energy holds what it does not use", free_size(energy(p)), least_size(energy(p)));
  }
  on_a_full_device("rif_build on a full device", build(RIF_FP64));
  on_a_full_device("pnof_energy_grad on a full device", energy(RIF_FP64));
  // a batch has an arena of its own: as large as its molecules' smallest
  for (rif_prec p : {RIF_FP64, RIF_FP32, RIF_BF16X6}) {
    const rif_instance two[] = {in, in};
    const size_t least = (least_size(build(p)) + 255) / 256 * 256;
    rif_ctx c;
    rif_batch* bt = nullptr;
    device_free = 2 * least;
    check(rif_batch_create(&c, 2, two, p, RIF_PNOF7, &bt) == RIF_OK, "batch on a full device", 2 * least);
    if (bt) {
      check(rif_batch_run(bt, 0) == RIF_OK, "batch on a full device runs");
      rif_batch_destroy(bt);
    }
    device_free = ~size_t(0);
  }
}

// The network's backward pass runs in the gradients at its logits and one double
// for every 256 rows.
static void training() {
  for (int rows : {1, 40, 257, 4096, 6001, 13001, 100003}) {
    float x = 0.f;
    auto back = [&](rif_ctx* c) { return rif_mlp_backward(c, rows, &x, &x, &x, &x, &x, &x, &x, &x, &word); };
    const size_t need = ((rows + 255) / 256 * sizeof(double) + 255) / 256 * 256 + (size_t)rows * 7 * sizeof(float);
    check(runs_with(need, back), "rif_mlp_backward", rows, need);
    on_a_full_device("rif_mlp_backward on a full device", back);
  }
}

// The preparation runs column by column in six n_aux^2 matrices, with the packed
// triangles' n_aux n_bf (n_bf + 1) / 2 to spare.
static void preparation() {
  for (int n : {40, 1044, 1601, 1800, 2048, 2049})
    for (int nb : {1, 12, 60}) {
      auto prep = [&](rif_ctx* c) { return rif_prepare_b(c, nb, n, &word, &word, 0.0, &word, nullptr, nullptr, nullptr, nullptr); };
      const size_t nn = (size_t)n * n, need = 8 * (6 * nn + 2 * (size_t)n + (size_t)n * nb * (nb + 1) / 2) + 12 * 256;
      check(runs_with(need, prep), "rif_prepare_b", n, nb);
      if (n > 400) on_a_full_device("rif_prepare_b on a full device", prep);
    }
}

// A program that loads tile choices saved by an earlier version (four FP64 variants a
// step, the Fock step's splits in its key) and captures its build after a first run.
static void saved_choices() {
  const rif_instance in = molecule(348, 1044, 24, 4, 348);
  const char* saved =
      "half_transform 0 348 363312 120 348 -> 2 | 0.60 0.62 0.58 0.61\n"
      "mo_transform 0 348 1044 120 348 -> 3 | 0.22 0.25 0.24 0.21\n"
      "jao 0 348 1044 120 -> 3 | 0.31 0.33 0.32 0.30\n"
      "kao 0 348 1044 120 -> 1 | 0.35 0.33\n"
      "fock 0 348 120 348 42 -> 0 | 0.16 0.18 0.17 0.17\n";
  rif_ctx c;
  check(rif_tune_load(&c, saved) == RIF_OK, "saved choices load");
  check(rif_build(&c, &in, RIF_FP64, RIF_PNOF7) == RIF_OK, "first build");   // the arena
  c.tune_mode = 1;
  capturing = true;
  check(rif_build(&c, &in, RIF_FP64, RIF_PNOF7) == RIF_OK, "captured build with saved choices");
  capturing = false;
  const size_t launches = n_launch;
  check(rif_build(&c, &in, RIF_FP64, RIF_PNOF7) == RIF_OK && n_launch > launches, "build after it");
}

int main() {
  builds();
  training();
  preparation();
  saved_choices();
  printf("%d checks, %d failures\n", n_check, n_fail);
  return n_fail != 0;
}
