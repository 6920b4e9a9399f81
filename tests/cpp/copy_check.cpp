// Host-only check of the copy of results to the caller (host_copy.cpp), built
// against the HIP headers with the runtime's functions defined here on host
// memory: a copy is done at once.
// Arguments: the device of the stream (device 0 is current; an event made on one device
// is refused on the stream of another), then lengths in bytes.  For each, a piece of that many bytes and two
// short ones are copied into arrays filled with a sentinel; prints one line
// "len=... bad=..." with the number of bytes that did not arrive.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "internal.hpp"

int cosm::set_error(int st, const std::string &m) { fprintf(stderr, "err %s\n", m.c_str()); return st; }
void cosm::clear_error() {}

// a stream is its device + 1, an event lives on device 0
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
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  memcpy(d, s, n);
  return hipSuccess;
}
}

int main(int argc, char **argv) {
  if (argc < 2) return 1;
  const hipStream_t stream = (hipStream_t)(intptr_t)(atoi(argv[1]) + 1);
  for (int i = 2; i < argc; i++) {
    const size_t len = strtoull(argv[i], nullptr, 10), small = 800;
    std::vector<unsigned char> src(len + 2 * small), a(len + 64, 0xee), b(small, 0xee), c(small, 0xee);
    for (size_t k = 0; k < src.size(); k++) src[k] = (unsigned char)(k * 131 % 199);  // never 0xee
    cosm::HostPiece p[cosm::kHostPieces] = {{b.data(), src.data() + len, small},
                                            {c.data(), src.data() + len + small, small},
                                            {a.data(), src.data(), len}};
    const int rc = cosm::copy_to_host(stream, p, 3, true);
    size_t bad = rc != 0;
    for (size_t k = 0; k < len; k++) bad += a[k] != src[k];
    for (size_t k = len; k < a.size(); k++) bad += a[k] != 0xee;  // nothing past the array
    bad += memcmp(b.data(), src.data() + len, small) != 0;
    bad += memcmp(c.data(), src.data() + len + small, small) != 0;
    printf("len=%zu bad=%zu\n", len, bad);
  }
  return 0;
}
