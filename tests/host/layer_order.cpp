// The host runtime over a model of HIP's streams and events: every enqueued
// piece of work gets a vector clock (the work it is ordered after), so that
// what a launch reads or overwrites can be checked against what it must
// follow, and any HIP call can be made to fail.  runtime.hip is compiled as it
// stands; the kernel launchers and the HIP functions it calls are below.
#include <hip/hip_runtime.h>

#define HIP_SYMBOL(x) &(x)
#define __align__(n) __attribute__((aligned(n)))
#include "runtime.hip"

#include <algorithm>
#include <cstdlib>
#include <map>
#include <set>

// ---------------------------------------------------------------- the model
namespace {

using Clock = std::set<int>;  // ids of the pieces of work something is ordered after
struct Stream { Clock after; };
struct Event { Clock after; };
Stream null_stream;
int n_work = 0;
int fail_at = -1, n_calls = 0;  // fail the fail_at-th call that may fail

Stream *S(hipStream_t s) { return s ? reinterpret_cast<Stream *>(s) : &null_stream; }
Event *V(hipEvent_t e) { return reinterpret_cast<Event *>(e); }
bool fails() { return n_calls++ == fail_at; }
int work(hipStream_t s) {
  const int id = n_work++;
  S(s)->after.insert(id);
  return id;
}
[[noreturn]] void die(const char *what) {
  std::printf("%s\n", what);
  std::exit(1);
}
// every piece of work in `ids` is ordered before what stream s runs next
void must_follow(hipStream_t s, const Clock &ids, const char *what) {
  for (const int i : ids)
    if (!S(s)->after.count(i)) die(what);
}

// who last used each buffer: arena readers and writers, per-slot scratch
Clock arena_users;               // staging and batch work of earlier layers
Clock layer_users;               // of the open layer
std::map<const void *, Clock> scratch_users;
std::set<int> staged_ids;        // arena rows whose ids this layer's staging wrote
int batches_routed = 0;

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipMalloc(void **p, size_t) { return *p = std::malloc(64), hipSuccess; }
hipError_t hipFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
  if (fails()) return hipErrorOutOfMemory;
  return *p = std::calloc(1, n), hipSuccess;
}
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) {
  return *p = const_cast<void *>(s), hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
  return *s = reinterpret_cast<hipStream_t>(new Stream), hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { return delete S(s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
  return *e = reinterpret_cast<hipEvent_t>(new Event), hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { return delete V(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  if (fails()) return hipErrorUnknown;
  return V(e)->after = S(s)->after, hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  if (fails()) return hipErrorUnknown;
  S(s)->after.insert(V(e)->after.begin(), V(e)->after.end());
  return hipSuccess;
}
// nothing has finished yet: the case that needs every order to be stated
hipError_t hipEventQuery(hipEvent_t) { return hipErrorNotReady; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *t, hipEvent_t, hipEvent_t) { return *t = 0, hipSuccess; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t s) {
  if (fails()) return hipErrorUnknown;
  return work(s), hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *, size_t n, hipMemcpyKind) {
  return std::memset(d, 0, n), hipSuccess;
}
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}

// ------------------------------------------------------------ the launchers
namespace cep {

hipError_t launch_pack_w1(const void *, const void *, int, int, int, uint8_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_w2(const void *, int, int, int, uint8_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_scales(const float *, const float *, const float *, int, int, float *, float *, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_mx(const uint8_t *, const uint8_t *, const uint8_t *, const uint8_t *, const uint8_t *, const uint8_t *, int, int, uint8_t *, const BlobLayout &, hipStream_t) { return hipSuccess; }

static void use_arena(hipStream_t s) {
  must_follow(s, arena_users, "arena used before the previous layer's work on it");
  layer_users.insert(work(s));
}
static void use_scratch(const Scratch &sc, hipStream_t s) {
  Clock &u = scratch_users[sc.cnt];
  must_follow(s, u, "a slot's scratch used before its previous batch");
  u = {work(s)};
}

hipError_t launch_ingest(const Arena &, const IngestGroup &grp, int, int, int, size_t, uint32_t *,
                         hipStream_t s) {
  if (fails()) return hipErrorUnknown;
  use_arena(s);
  for (int i = 0; i < grp.n; ++i)
    for (int r = 0; r < grp.c[i].n_rows; ++r) staged_ids.insert(grp.c[i].row0 + r);
  return hipSuccess;
}
bool stage_in_route(const IngestGroup &grp, int row0, int n_rows, int k) {
  if (grp.n < 1 || grp.n > kStageChunks || (long long)n_rows * k > kFusedRoutePairs) return false;
  int r = row0;
  for (int i = 0; i < grp.n; ++i) {
    if (grp.c[i].row0 != r) return false;
    r += grp.c[i].n_rows;
  }
  return r == row0 + n_rows;
}
hipError_t launch_route(const Arena &, const Scratch &sc, const IngestGroup *stage, int, size_t,
                        int row0, int n_rows, int k, int, int, int, int, int, uint64_t, int, int,
                        int, int, int, int, uint32_t *, hipStream_t s) {
  if (fails()) return hipErrorUnknown;
  if (stage && !stage_in_route(*stage, row0, n_rows, k)) return hipErrorInvalidValue;
  // without chunks to stage the kernel reads the arena's ids
  for (int r = row0; !stage && r < row0 + n_rows; ++r)
    if (!staged_ids.count(r)) die("routing reads arena ids that nothing staged");
  use_arena(s);
  use_scratch(sc, s);
  ++batches_routed;
  return hipSuccess;
}
hipError_t launch_gemm1(const Scratch &sc, int, int, int, int, int, int, const BlobTable &,
                        const BlobLayout &, int, int, int, const Arena *, int, int, hipStream_t s) {
  if (fails()) return hipErrorUnknown;
  use_arena(s);
  use_scratch(sc, s);
  return hipSuccess;
}
hipError_t launch_gemm2(const Scratch &sc, int, int, int, int, int, int, const BlobTable &,
                        const BlobLayout &, int, int, int, float *, hipStream_t s) {
  if (fails()) return hipErrorUnknown;
  use_scratch(sc, s);
  return hipSuccess;
}
hipError_t launch_combine(const Arena &, const Scratch &sc, int, int, int, int, bool, bool, float *,
                          hipStream_t s) {
  if (fails()) return hipErrorUnknown;
  use_arena(s);
  use_scratch(sc, s);
  return hipSuccess;
}

}  // namespace cep

// ------------------------------------------------------------------- checks
namespace {

unsigned long long seed = 1;
int rnd(int n) {
  seed = seed * 6364136223846793005ull + 1442695040888963407ull;
  return (int)((seed >> 33) % (unsigned)n);
}

int ints[1];
float floats[1];
alignas(16) float rows16[4];

cep_ctx *make(int streams, int record) {
  cep_config cfg{};
  cfg.d_model = 256, cfg.d_ff = 128, cfg.n_local_experts = 4, cfg.top_k = 2;
  cfg.max_replicas = 2, cfg.max_tokens_per_replica = 8192;
  cfg.w_dtype = CEP_BF16, cfg.x_dtype = CEP_BF16;
  cfg.n_streams = streams, cfg.record_routing = record;
  cep_weights w{floats, floats, floats, nullptr, nullptr, nullptr};
  cep_ctx *c = nullptr;
  if (cep_init_experts(&c, &cfg, &w, nullptr, nullptr) != CEP_OK) die(cep_last_error(nullptr));
  return c;
}

int submit(cep_ctx *c, uint32_t gen, int n_rows, int n_pairs, hipEvent_t arrival) {
  return cep_submit_chunk(c, gen, 0, n_rows, n_pairs, ints, rows16, ints, floats, arrival, nullptr);
}

// One layer of random chunks under a random policy, no synchronisation before
// or after; every call succeeds.
void layer(cep_ctx *c, uint32_t gen, int max_streams, hipStream_t s) {
  const int policies[] = {CEP_WAIT_ALL, CEP_PER_CHUNK, CEP_THRESHOLD};
  if (cep_set_policy(c, policies[rnd(3)], 1 + rnd(600), 1 + rnd(max_streams)) != CEP_OK)
    die(cep_last_error(c));
  const int n = rnd(7);
  if (cep_begin_layer(c, gen, 1, &n, floats) != CEP_OK) die(cep_last_error(c));
  staged_ids.clear();
  layer_users.clear();
  for (int i = 0; i < n; ++i) {
    const int n_rows = rnd(4) ? rnd(4) == 0 ? 1 + rnd(2500) : 1 + rnd(300) : 0;
    const int n_pairs = rnd(3) ? rnd(2 * n_rows + 1) : 0;
    Event arrived{{work(nullptr)}};
    const bool wait = rnd(2);
    if (submit(c, gen, n_rows, n_pairs, wait ? reinterpret_cast<hipEvent_t>(&arrived) : nullptr) !=
        CEP_OK)
      die(cep_last_error(c));
    if (rnd(6) == 0 && cep_flush(c) != CEP_OK) die(cep_last_error(c));
  }
  hipEvent_t done = nullptr;
  if (cep_combine(c, s, &done) != CEP_OK) die(cep_last_error(c));
  for (const int i : layer_users)
    if (!V(done)->after.count(i)) die("done is not ordered after the layer's work");
  arena_users = layer_users;
}

void orders() {
  for (int it = 0; it < 300; ++it) {
    const int ns = 1 + rnd(4);
    cep_ctx *c = make(ns, rnd(2));
    Stream caller;
    arena_users.clear();
    for (int g = 1; g <= 8; ++g) layer(c, g, ns, reinterpret_cast<hipStream_t>(&caller));
    cep_destroy(c);
    scratch_users.clear();
  }
}

// A batch whose launch fails at its n-th step stays pending, and a flush runs
// it whole.
void retries() {
  for (int record = 0; record < 2; ++record)
    for (int rows : {40, 3000}) {  // staged by the routing launch, by a launch of its own
      int failed = 0;
      for (int n = 0; n < 40; ++n) {
        cep_ctx *c = make(2, record);
        arena_users.clear(), scratch_users.clear(), staged_ids.clear();
        if (cep_set_policy(c, CEP_PER_CHUNK, 1, 2) != CEP_OK) die(cep_last_error(c));
        const int chunks = 1;
        if (cep_begin_layer(c, 1, 1, &chunks, floats) != CEP_OK) die(cep_last_error(c));
        n_calls = 0, fail_at = n, batches_routed = 0;
        const int rc = submit(c, 1, rows, rows, nullptr);
        fail_at = -1;
        if (rc != CEP_OK) {
          ++failed;
          if (rc != CEP_EHIP || cep_get_batch_count(c) != 0) die("a failed launch left a batch");
          batches_routed = 0;
          if (cep_flush(c) != CEP_OK) die(cep_last_error(c));
        }
        if (batches_routed != 1 || cep_get_batch_count(c) != 1) die("the batch did not run");
        if (cep_combine(c, nullptr, nullptr) != CEP_OK) die(cep_last_error(c));
        cep_destroy(c);
      }
      if (failed < 5) die("no step failed");
    }
}

}  // namespace

int main() {
  orders();
  retries();
  return 0;
}
