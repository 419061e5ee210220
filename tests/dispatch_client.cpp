// A client of the C ABI that stands in for the device runtime's launch call: job lists and single calls go
// through the library's checks and its dispatch, and every launch is printed instead of made (the pointers
// are never followed).  Job: kind,dtype,bits,rounding,batch,n_per,group.  Options: "alone" makes each job a
// call of its own, "lowbit" decodes with previous messages kept at 8 bits; "starve" lets every allocation fail once something has been launched.
#include <dlfcn.h>
#include <cxxabi.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "aqsgd.h"

static int g_launches = 0;
static bool g_starve = false;

void* operator new(std::size_t n) {
    if (g_starve && g_launches > 0) throw std::bad_alloc();
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

extern "C" hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void**, size_t, hipStream_t) {
    Dl_info info = {};
    char* name = nullptr;
    if (dladdr(f, &info) && info.dli_sname) name = abi::__cxa_demangle(info.dli_sname, nullptr, nullptr, nullptr);
    std::printf("launch %u %u %u x %u %s\n", grid.x, grid.y, grid.z, block.x, name ? name : "?");
    std::free(name);
    ++g_launches;
    return hipSuccess;
}

int main(int argc, char** argv) {
    bool alone = false, lowbit = false;
    std::vector<aqsgd_job> jobs;
    for (int i = 1; i < argc; ++i) {
        if (!std::strcmp(argv[i], "alone")) { alone = true; continue; }
        if (!std::strcmp(argv[i], "lowbit")) { lowbit = true; continue; }
        if (!std::strcmp(argv[i], "starve")) { g_starve = true; continue; }
        int kind, dtype, bits, rounding;
        long batch, n_per;
        int group;
        if (std::sscanf(argv[i], "%d,%d,%d,%d,%ld,%ld,%d", &kind, &dtype, &bits, &rounding, &batch, &n_per, &group) != 7) return 2;
        aqsgd_job j;
        std::memset(&j, 0, sizeof j);
        j.kind = static_cast<decltype(j.kind)>(kind);
        j.desc.batch = batch; j.desc.n_per = n_per; j.desc.n_samples = 2 * batch; j.desc.bits = bits; j.desc.group = group;
        j.desc.dtype = static_cast<decltype(j.desc.dtype)>(dtype);
        j.desc.rounding = static_cast<decltype(j.desc.rounding)>(rounding);
        char* at = reinterpret_cast<char*>(uintptr_t{1} << 20);
        j.src = at; j.out = at; j.m_buf = at; j.sample_ids = reinterpret_cast<int64_t*>(at);
        j.codes = reinterpret_cast<uint8_t*>(at); j.scales = reinterpret_cast<float*>(at);
        jobs.push_back(j);
    }
    int status = 0;
    if (lowbit) {
        for (aqsgd_job& j : jobs) {
            status = aqsgd_decode_lowbit(&j.desc, 8, j.codes, j.scales, j.sample_ids, static_cast<uint8_t*>(j.m_buf), j.scales,
                                         j.out, nullptr);
            if (status) break;
        }
    } else if (alone) {
        for (aqsgd_job& j : jobs) {
            switch (j.kind) {
            case AQSGD_JOB_ENCODE: status = aqsgd_encode(&j.desc, j.src, j.sample_ids, j.m_buf, j.codes, j.scales, nullptr); break;
            case AQSGD_JOB_DECODE: status = aqsgd_decode(&j.desc, j.codes, j.scales, j.sample_ids, j.m_buf, j.out, nullptr); break;
            case AQSGD_JOB_GRAD_QUANT: status = aqsgd_grad_quant(&j.desc, j.src, j.codes, j.scales, nullptr); break;
            default: status = aqsgd_grad_dequant(&j.desc, j.codes, j.scales, j.out, nullptr); break;
            }
            if (status) break;
        }
    } else {
        status = aqsgd_run_jobs(jobs.data(), static_cast<int>(jobs.size()), nullptr);
    }
    std::printf("status %d\n", status);
    return 0;
}
