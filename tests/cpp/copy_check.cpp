// Host-only check of the copy of results to the caller (host_copy.cpp), built
// against the HIP headers with the runtime's functions defined here on host
// memory: a copy is done at once.
// Arguments: the device of the stream (device 0 is current; an event made on one device
// is refused on the stream of another), the milliseconds that the device works before
// anything arrives, then lengths in bytes.  For each, a piece of that many bytes and two
// short ones are copied into arrays filled with a sentinel; prints one line
// "len=... bad=... cpu_ms=..." with the number of bytes that did not arrive and the
// processor time that the process took for it.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <chrono>
#include <ctime>
#include <thread>
#include <vector>

#include "internal.hpp"

int cosm::set_error(int st, const std::string &m) { fprintf(stderr, "err %s\n", m.c_str()); return st; }
void cosm::clear_error() {}

// a stream is its device + 1, an event lives on device 0
static int busy_ms = 0;
static bool busy = false;
static hipError_t arrive() {  // (waits asleep, so that only the copy's own threads can burn time)
  if (busy) std::this_thread::sleep_for(std::chrono::milliseconds(busy_ms));
  busy = false;
  return hipSuccess;
}
static int stream_device(hipStream_t s) { return (int)(intptr_t)s - 1; }

extern "C" {
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t *d) { *d = stream_device(s); return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = malloc(n); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t s) {
  return stream_device(s) == 0 ? hipSuccess : hipErrorInvalidHandle;
}
hipError_t hipStreamQuery(hipStream_t) { return busy ? hipErrorNotReady : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return arrive(); }
hipError_t hipStreamSynchronize(hipStream_t) { return arrive(); }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  return hipSuccess;
}
}

int main(int argc, char **argv) {
  if (argc < 3) return 1;
  busy_ms = atoi(argv[2]);
  const hipStream_t stream = (hipStream_t)(intptr_t)(atoi(argv[1]) + 1);
  for (int i = 3; i < argc; i++) {
    const size_t len = strtoull(argv[i], nullptr, 10), small = 800;
    std::vector<unsigned char> src(len + 2 * small), a(len + 64, 0xee), b(small, 0xee), c(small, 0xee);
    for (size_t k = 0; k < src.size(); k++) src[k] = (unsigned char)(k * 131 % 199);  // never 0xee
    cosm::HostPiece p[cosm::kHostPieces] = {{b.data(), src.data() + len, small},
                                            {c.data(), src.data() + len + small, small},
                                            {a.data(), src.data(), len}};
    busy = true;
    const clock_t t0 = clock();
    const int rc = cosm::copy_to_host(stream, p, 3, true);
    const double cpu_ms = 1000.0 * (double)(clock() - t0) / CLOCKS_PER_SEC;
    size_t bad = rc != 0;
    for (size_t k = 0; k < len; k++) bad += a[k] != src[k];
    for (size_t k = len; k < a.size(); k++) bad += a[k] != 0xee;  // nothing past the array
    bad += memcmp(b.data(), src.data() + len, small) != 0;
    bad += memcmp(c.data(), src.data() + len + small, small) != 0;
    printf("len=%zu bad=%zu cpu_ms=%.1f\n", len, bad, cpu_ms);
  }
  return 0;
}
