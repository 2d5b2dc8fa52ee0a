// A stand-in for the HIP runtime for tests of the library's host code on a
// machine without a GPU: device memory is host memory, kernels do nothing, and
// streams, events, captures and executable graphs are tracked.  Misuse (a
// graph destroyed while a launch of it may still run, an event of an ended
// capture waited for, a stream left unjoined by a capture, copies or fills in
// a capture, work issued while another device is current, launches out of the
// documented limits) is counted and printed.
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>

namespace {

struct Capture {
  void* origin;
  bool active;
  std::set<void*> streams, open;
};
struct Stream {
  Capture* cap = nullptr;
  std::set<void*> in_flight;  // graphs launched since the stream was last waited for
};
struct Event {
  Capture* cap = nullptr;
  void* stream = nullptr;
  bool recorded = false;
};
struct dim3 {
  unsigned x, y, z;
};
struct {
  dim3 g, b;
  size_t lds;
  void* s;
} pushed;
struct All {
  std::set<void*> streams, events, graphs, execs;
  Stream null;
  int misuses = 0, device = 0;
};
All& all() {
  static All* a = new All;  // (the library's static constructors come first)
  return *a;
}
void misuse(const char* f, ...) {
  va_list v;
  va_start(v, f);
  printf("misuse: ");
  vprintf(f, v);
  printf("\n");
  va_end(v);
  ++all().misuses;
}
template <class T>
T* known(std::set<void*>& s, void* p, const char* what) {
  if (!s.count(p)) {
    misuse("unknown %s", what);
    fflush(stdout);
    exit(3);
  }
  return static_cast<T*>(p);
}
// (every context of the tests is on device 0)
void on_device(const char* what) {
  if (all().device != 0) misuse("%s with another device current", what);
}
Stream* stream_of(void* s) { return s ? known<Stream>(all().streams, s, "stream") : &all().null; }

}  // namespace

extern "C" {

int stub_misuses() {
  fflush(stdout);
  return all().misuses;
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void* s) {
  pushed = {g, b, lds, s};
  return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, void** s) {
  *g = pushed.g;
  *b = pushed.b;
  *lds = pushed.lds;
  *s = pushed.s;
  return 0;
}
void** __hipRegisterFatBinary(const void*) {
  static void* p;
  return &p;
}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
int hipDeviceGetAttribute(int* v, int, int) {
  *v = 163840;
  return 0;
}
int hipSetDevice(int d) {
  all().device = d;
  return 0;
}
int hipGetDevice(int* d) {
  *d = all().device;
  return 0;
}
int hipGetDeviceCount(int* d) {
  *d = 2;
  return 0;
}
const char* hipGetErrorString(int) { return "error"; }
int hipGetLastError() { return 0; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = malloc(64 << 20);
  *p = scratch;
  return 0;
}
int hipMalloc(void** p, size_t n) {
  on_device("allocation");
  *p = malloc(n);
  if (*p) memset(*p, 0xa5, n);
  return *p ? 0 : 2;
}
int hipFree(void* p) {
  free(p);
  return 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int) {
  on_device("copy");
  if (n) memcpy(d, s, n);
  return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void* st) {
  on_device("copy");
  if (stream_of(st)->cap) misuse("copy in a capture");
  if (n) memcpy(d, s, n);
  return 0;
}
int hipMemset(void* d, int v, size_t n) {
  on_device("fill");
  memset(d, v, n);
  return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void* st) {
  on_device("fill");
  if (stream_of(st)->cap) misuse("fill in a capture");
  memset(d, v, n);
  return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned) {
  all().streams.insert(*s = new Stream);
  return 0;
}
int hipStreamDestroy(void* s) {
  Stream* t = known<Stream>(all().streams, s, "stream");
  all().streams.erase(s);
  delete t;
  return 0;
}
int hipStreamSynchronize(void* s) {
  if (stream_of(s)->cap) misuse("wait in a capture");
  stream_of(s)->in_flight.clear();
  return 0;
}
int hipEventCreateWithFlags(void** e, unsigned) {
  all().events.insert(*e = new Event);
  return 0;
}
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void* e) {
  Event* t = known<Event>(all().events, e, "event");
  all().events.erase(e);
  delete t;
  return 0;
}
int hipEventRecord(void* e, void* s) {
  Event* x = known<Event>(all().events, e, "event");
  x->cap = stream_of(s)->cap;
  x->stream = s;
  x->recorded = true;
  return 0;
}
int hipEventSynchronize(void* e) {
  Event* x = known<Event>(all().events, e, "event");
  if (x->cap)
    misuse("wait for a captured event");
  else
    stream_of(x->stream)->in_flight.clear();
  return 0;
}
int hipEventElapsedTime(float* ms, void*, void*) {
  *ms = 1.0f;
  return 0;
}
int hipStreamWaitEvent(void* s, void* e, unsigned) {
  Event* x = known<Event>(all().events, e, "event");
  Stream* t = stream_of(s);
  if (!x->recorded) misuse("wait for an event that was never recorded");
  if (!x->cap) {
    if (t->cap) misuse("a captured stream waits for an event of none");
    return 0;
  }
  if (!x->cap->active) misuse("wait for an event of an ended capture");
  if (t->cap && t->cap != x->cap) misuse("two captures joined");
  t->cap = x->cap;
  t->cap->streams.insert(s);
  if (s == x->cap->origin)
    x->cap->open.erase(x->stream);
  else
    x->cap->open.insert(s);
  return 0;
}
int hipStreamBeginCapture(void* s, int) {
  on_device("capture");
  Stream* t = stream_of(s);
  if (t->cap) misuse("capture in a capture");
  t->cap = new Capture{s, true, {s}, {}};
  return 0;
}
int hipStreamEndCapture(void* s, void** g) {
  Capture* c = stream_of(s)->cap;
  if (!c || c->origin != s) {
    misuse("end of no capture");
    return 1;
  }
  if (!c->open.empty()) misuse("a stream of the capture is not joined");
  c->active = false;  // (kept: events may still name it)
  for (void* x : c->streams) static_cast<Stream*>(x)->cap = nullptr;
  all().graphs.insert(*g = new char);
  return 0;
}
int hipGraphInstantiate(void** x, void* g, void**, char*, size_t) {
  on_device("instantiation");
  known<char>(all().graphs, g, "graph");
  all().execs.insert(*x = new char);
  return 0;
}
int hipGraphDestroy(void* g) {
  delete known<char>(all().graphs, g, "graph");
  all().graphs.erase(g);
  return 0;
}
int hipGraphLaunch(void* x, void* s) {
  on_device("graph launch");
  known<char>(all().execs, x, "executable graph");
  stream_of(s)->in_flight.insert(x);
  return 0;
}
int hipGraphExecDestroy(void* x) {
  char* p = known<char>(all().execs, x, "executable graph");
  for (void* s : all().streams)
    if (static_cast<Stream*>(s)->in_flight.count(x)) misuse("a graph destroyed in flight");
  all().execs.erase(x);
  delete p;
  return 0;
}
int hipLaunchKernel(const void*, dim3 g, dim3 b, void**, size_t lds, void* s) {
  on_device("launch");
  Stream* t = stream_of(s);
  if (!g.x || !g.y || !g.z || !b.x || b.x * b.y * b.z > 1024 || lds > 163840)
    misuse("launch of %u x %u blocks of %u threads with %zu bytes of LDS", g.x, g.y, b.x, lds);
  if (t->cap && s != t->cap->origin) t->cap->open.insert(s);
  return 0;
}
}
