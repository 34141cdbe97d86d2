// A HIP runtime that only keeps a log: preloaded in front of libamdhip64, it
// lets the built library's host code (which form a call takes, on which
// streams, with which waits) run without a GPU. Copies are done on host memory,
// kernels are noted by name, and the time between two events is the number of
// kernels between them. dry_fail(text): launches of kernels whose name holds
// `text` fail from then on ("": none).
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
std::string log_text, fail_name;
std::map<const void *, std::string> kernels;
std::map<void *, int> event_time;
int last_error = 0, launches = 0, capture_status = 0;
uintptr_t next_handle = 1;

void note(const char *what, void *stream, const std::string &rest)
{
    char head[64];
    snprintf(head, sizeof head, "%s %d ", what, (int)(uintptr_t)stream);
    log_text += head + rest + "\n";
}

int launch(const char *what, const void *f, unsigned gx, unsigned gy, void *stream, void **args = nullptr)
{
    const std::string &name = kernels[f];
    if (!fail_name.empty() && name.find(fail_name) != std::string::npos)
        return last_error = 2;   // hipErrorOutOfMemory
    ++launches;
    const bool fill = args && name.find("k_fill_u32") != std::string::npos;   // (its number of words)
    note(what, stream, name + " " + std::to_string(gx) + " " + std::to_string(gy) +
                           (fill ? " " + std::to_string(*(const size_t *)args[1]) : ""));
    return 0;
}

int fresh(void **out)
{
    *out = (void *)next_handle++;
    return 0;
}

struct Dim { unsigned x, y, z; };
struct Config { Dim grid, block; size_t shared; void *stream; };
std::vector<Config> configs;
}  // namespace

extern "C" {
const char *dry_log() { return log_text.c_str(); }
void dry_clear() { log_text.clear(); }
void dry_fail(const char *text) { fail_name = text; }
void dry_capturing(int on) { capture_status = on; }

void **__hipRegisterFatBinary(const void *) { static void *m; return &m; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { kernels[f] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim g, Dim b, size_t shared, void *s) { configs.push_back({g, b, shared, s}); return 0; }
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *shared, void **s)
{
    const Config c = configs.back();
    configs.pop_back();
    *g = c.grid; *b = c.block; *shared = c.shared; *s = c.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim g, Dim, void **args, size_t, void *s) { return launch("launch", f, g.x, g.y, s, args); }
int hipLaunchCooperativeKernel(const void *f, Dim g, Dim, void **, unsigned, void *s) { return launch("launch", f, g.x, g.y, s); }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int e) { return e == 0 ? "no error" : e == 2 ? "out of memory" : "some error"; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { *n = 1; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipGetSymbolAddress(void **, const void *) { return 1; }
int hipMemcpy(void *d, const void *s, size_t n, int) { memcpy(d, s, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int, void *) { memcpy(d, s, n); return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { return fresh(s); }
int hipStreamDestroy(void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned) { note("wait", s, std::to_string((uintptr_t)e)); return 0; }
int hipStreamIsCapturing(void *, int *status) { *status = capture_status; return 0; }
int hipStreamBeginCapture(void *s, int) { note("capture", s, ""); return 0; }
int hipStreamEndCapture(void *s, void **g) { note("captured", s, ""); return fresh(g); }
int hipGraphInstantiate(void **x, void *, void **, char *, size_t) { return fresh(x); }
int hipGraphLaunch(void *, void *s) { note("graph", s, ""); return 0; }
int hipGraphDestroy(void *) { return 0; }
int hipGraphExecDestroy(void *) { return 0; }
int hipEventCreate(void **e) { return fresh(e); }
int hipEventCreateWithFlags(void **e, unsigned) { return fresh(e); }
int hipEventDestroy(void *) { return 0; }
int hipEventRecord(void *e, void *s) { event_time[e] = launches; note("record", s, std::to_string((uintptr_t)e)); return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { *ms = (float)(event_time[b] - event_time[a]); return 0; }
}
