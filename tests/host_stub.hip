// Stand-ins for the HIP runtime and the kernel launchers, for tests of the library's host code without a GPU: zp_api.hip and
// zp_kernels.hip are compiled for the host only and linked against this file.  Nothing is launched; every call is written to a log.
#include "../paper_2603_08743_amd/csrc/zp_kernels.h"

#include <cstdarg>
#include <cstdio>
#include <map>
#include <string>

static std::string g_log;
static std::string g_attributes;              // kernels that were given the large LDS limit, since the library was loaded
static std::map<std::string, int> g_set;      // stub_set: device, stream_device, capturing, no_memory
static std::map<const void *, std::string> &names() {   // filled while the library is loaded, before this file's own variables exist
    static std::map<const void *, std::string> m;
    return m;
}
extern "C" { char stub_blob[64]; }

static void note(const char *fmt, ...) {
    char line[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(line, sizeof(line), fmt, ap);
    va_end(ap);
    g_log += line;
    g_log += "\n";
}

extern "C" {
const char *stub_log() { return g_log.c_str(); }
const char *stub_attributes() { return g_attributes.c_str(); }
void stub_clear() { g_log.clear(); }
void stub_set(const char *what, int value) { g_set[what] = value; }

hipError_t hipGetDevice(int *d) { *d = g_set["device"]; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t *d) { *d = g_set["stream_device"]; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) {
    if (g_set["no_memory"] && n > 4096) return hipErrorOutOfMemory;
    *p = (void *)((uintptr_t)0x700000000000 + (n > 4096 ? 0x1000000 : 0));
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { static char mem[4096]; *p = mem; return n <= sizeof(mem) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { return hipErrorInvalidValue; }
hipError_t hipMemcpyAsync(void *, const void *, size_t, hipMemcpyKind, hipStream_t) { return hipErrorInvalidValue; }
hipError_t hipFree(void *) { return hipSuccess; }
hipError_t hipHostFree(void *) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = stub_blob; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v) { g_attributes += names()[f] + " " + std::to_string(v) + "\n"; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c) {
    *c = g_set["capturing"] ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { static uintptr_t n = 0; *e = (hipEvent_t)++n; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { note("record %d stream %d", (int)(uintptr_t)e, (int)(uintptr_t)s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { note("wait %d stream %d", (int)(uintptr_t)e, (int)(uintptr_t)s); return hipSuccess; }

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names()[host] = name; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *n, hipStream_t *s) { *g = *b = dim3(1); *n = 0; *s = nullptr; return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t) {
    const std::string &name = names()[f];
    if (name.find("unit_") == std::string::npos) { note("launch %s", name.c_str()); return hipSuccess; }
    const zp::Args &a = *(const zp::Args *)args[0];
    note("launch %s units %d stages %d slices %d slice_bytes %d lds %d fixed %d", name.find("sliced") != std::string::npos ? "unit_sliced" : "unit_generic",
         a.B * a.L_slab * a.h_kv, a.stages, a.slices, a.slice_bytes, a.lds_bytes, a.unit_in != nullptr);
    return hipSuccess;
}
}  // extern "C"

namespace zp {
static hipError_t mfma(const Args &a, int units, int NW) {
    note("launch unit_mfma units %d stages %d phase %d parts %d NW %d lds %d", units, a.stages, a.phase, a.parts, NW, a.lds_bytes);
    return hipSuccess;
}
#define ZP_STUB_MFMA(name) hipError_t name(const Args &a, int units, int NW, int, hipStream_t) { return mfma(a, units, NW); }
ZP_STUB_MFMA(launch_mfma_d64) ZP_STUB_MFMA(launch_mfma_d64_wide) ZP_STUB_MFMA(launch_mfma_d64_ref) ZP_STUB_MFMA(launch_mfma_d64_wide_ref)
ZP_STUB_MFMA(launch_mfma_d128) ZP_STUB_MFMA(launch_mfma_d128_wide) ZP_STUB_MFMA(launch_mfma_d128_ref) ZP_STUB_MFMA(launch_mfma_d128_wide_ref)
ZP_STUB_MFMA(launch_mfma_pad_bf16) ZP_STUB_MFMA(launch_mfma_pad_bf16_long) ZP_STUB_MFMA(launch_mfma_pad_f32)
hipError_t launch_decode_attention(const DecodeArgs &, int, hipStream_t) { return hipSuccess; }
}  // namespace zp
