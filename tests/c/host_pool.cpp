// The library's device memory pool on a device of a few megabytes that only counts: the HIP
// calls below stand in for the runtime.  Built with the pool's own source.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <random>

#include "host_copy.hip"

static size_t g_free = 0;             // bytes the device still has
static std::map<void*, size_t> g_live;  // its allocations

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
    if (n > g_free) return hipErrorOutOfMemory;
    *p = aligned_alloc(256, (n + 255) / 256 * 256);
    g_live[*p] = n;
    g_free -= n;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    g_free += g_live.at(p);
    g_live.erase(p);
    free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
}
bool ccdk::alloc_injected() { return false; }

#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)

int main() {
    constexpr size_t MiB = size_t(1) << 20;
    void *a, *b, *c;
    {  // memory that the other pool holds without use serves this one
        g_free = 64 * MiB;
        ccdk::DevicePool kept, temp;
        kept.set_peer(&temp);
        temp.set_peer(&kept);
        temp.expect(48 * MiB);
        CHECK(temp.take(&a, 30 * MiB) == hipSuccess);
        temp.give(a);
        CHECK(temp.held() == 48 * MiB);
        CHECK(kept.take(&b, 40 * MiB) == hipSuccess);
        CHECK(temp.held() == 0 && kept.held() == 40 * MiB);
        // ... but not where it holds a block
        CHECK(temp.take(&a, 10 * MiB) == hipSuccess);
        CHECK(kept.take(&c, 30 * MiB) == hipErrorOutOfMemory && c == nullptr);
        CHECK(kept.take(&c, 10 * MiB) == hipSuccess);
        // A pool's own idle memory serves a larger block.
        kept.give(b);
        CHECK(kept.take(&b, 44 * MiB) == hipSuccess);
    }
    CHECK(g_live.empty());
    // Blocks do not overlap, and all memory is given back.
    std::mt19937_64 r(1);
    g_free = 96 * MiB;
    {
        ccdk::DevicePool pools[2];
        pools[0].set_peer(&pools[1]);
        pools[1].set_peer(&pools[0]);
        struct Block { char* p; size_t n; int pool; };
        std::vector<Block> v;
        int failed = 0;
        for (int it = 0; it < 100000; ++it) {
            if (v.size() < 120 && r() % 2) {
                const size_t n = (size_t(1) << (r() % 22)) + r() % 1000;
                const int k = (int)(r() % 2);
                void* p = nullptr;
                if (pools[k].take(&p, n) != hipSuccess) {
                    ++failed;
                    continue;
                }
                for (const Block& x : v) CHECK((char*)p + n <= x.p || x.p + x.n <= (char*)p);
                v.push_back({(char*)p, n, k});
            } else if (!v.empty()) {
                const size_t i = r() % v.size();
                pools[v[i].pool].give(v[i].p);
                v[i] = v.back();
                v.pop_back();
                if (r() % 100 == 0) pools[r() % 2].trim(r() % (32 * MiB));
            }
        }
        printf("failed takes: %d\n", failed);
    }
    CHECK(g_live.empty() && g_free == 96 * MiB);
    puts("ok");
    return 0;
}
