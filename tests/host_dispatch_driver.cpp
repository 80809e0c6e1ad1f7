// What the C entry points of the built library launch, without a GPU: this program defines the HIP runtime calls that the
// library makes (the dynamic linker prefers them to the runtime's), notes every kernel launch instead of making it, and
// prints which items each launch serves.  The items' x are made-up addresses that nothing reads; a launch's items
// are found by looking for them in its arguments.
//
// One list per line of standard input: "w4" or "w8", M, the number of items, then N, K and group size of each.  Answer:
// "list <status> <workspace asked for> <launches>", then one line per launch:
// "<kernel> <blocks> <workspace that its items ask for as a list of their own> <item> <item> ...", for the medium-batch kernel
// with the variants that its waves run after a bar, as "<column tiles>.<log2 of the K parts>".  First of all:
// "variants <mode>,<row blocks>,<column tiles>,<log2 of the K parts> ...", those that are compiled.
#include <cxxabi.h>
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <set>
#include <string>
#include <vector>

#include "midm_plan.h"

namespace {

constexpr uint64_t kX = 1ull << 52, kApart = 1ull << 36;   // item i's x lies at kX + i * kApart
constexpr int kMostItems = 512;

struct Launch {
    std::string kernel;
    unsigned blocks;
    std::vector<int> items;
    std::set<std::pair<int, int>> variants;
};
std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> m;
    return m;
}
std::vector<Launch> launches;
dim3 next_grid, next_block;
size_t next_lds;
hipStream_t next_stream;

// The records of the items stand first in a launch's only argument (or its arguments are a lone item's own).
size_t record_bytes(const std::string& kernel) {
    if (kernel.find("gemm_prep_kernel") != std::string::npos) return 8 * 56;
    if (kernel.find("midm_kernel") != std::string::npos) return sizeof(qail::MdArgs::it);
    if (kernel.find("smallm") != std::string::npos) return 16 * 64;
    return 0;
}

}  // namespace

extern "C" {

void** __hipRegisterFatBinary(const void*) {
    static void* module;
    return &module;
}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    int status = 0;
    char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    std::string s = status == 0 ? plain : name;
    free(plain);
    for (const char* cut : {"void ", "qail::", "(anonymous namespace)::", " "})
        for (size_t at; (at = s.find(cut)) != std::string::npos;) s.erase(at, strlen(cut));
    s = s.substr(0, s.find('('));
    names()[host] = s;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipUnregisterFatBinary(void**) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) {
    next_grid = grid;
    next_block = block;
    next_lds = lds;
    next_stream = st;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st) {
    *grid = next_grid;
    *block = next_block;
    *lds = next_lds;
    *st = next_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3, void** args, size_t, hipStream_t) {
    Launch l;
    l.kernel = names().count(f) ? names()[f] : "?";
    l.blocks = grid.x * grid.y * grid.z;
    std::vector<bool> seen(kMostItems);
    for (size_t at = 0; at + 8 <= record_bytes(l.kernel); at += 8) {
        uint64_t v;
        memcpy(&v, static_cast<const char*>(args[0]) + at, 8);
        if (v < kX || (v - kX) % kApart != 0 || (v - kX) / kApart >= kMostItems) continue;
        const int i = (int)((v - kX) / kApart);
        if (!seen[i]) l.items.push_back(i);
        seen[i] = true;
    }
    if (l.kernel.find("midm_kernel") != std::string::npos) {
        const qail::MdArgs& a = *static_cast<const qail::MdArgs*>(args[0]);
        for (const qail::MdItem& it : a.it)
            for (int more = 0; more < 2; ++more)   // blocks of tiles_base tiles and of one more
                for (int wave = 0; wave < qail::kMdWaves && (it.tiles_base + more > 0) && (more == 0 || it.tiles_rem > 0); ++wave)
                    l.variants.insert({std::max(1, qail::md_wave_tiles(it.tiles_base + more, it.wkl, wave)), it.wkl});
    }
    launches.push_back(l);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    memset(p, 0, sizeof(*p));
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorNotFound; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 1;
    return hipSuccess;
}

}  // extern "C"

int main(int argc, char** argv) {
    void* const so = argc == 2 ? dlopen(argv[1], RTLD_NOW | RTLD_GLOBAL) : nullptr;
    if (!so) {
        fprintf(stderr, "cannot load the library: %s\n", argc == 2 ? dlerror() : "no path given");
        return 1;
    }
#define FN(f) const auto f##_ = reinterpret_cast<decltype(&f)>(dlsym(so, #f))
    FN(qail_w4a16_batch_workspace);
    FN(qail_w4a16_linear_batch);
    FN(qail_w8a16_batch_workspace);
    FN(qail_w8a16_linear_batch);
#undef FN
    printf("variants");
    for (int mode = 0; mode < 3; ++mode)
        for (int rb = 1; rb <= 4; ++rb)
            for (int c = 1; c <= 4; ++c)
                for (int p = 0; p < 4; ++p)
                    if (qail::md_variant(mode, rb, c, p)) printf(" %d,%d,%d,%d", mode, rb, c, p);
    printf("\n");
    char kind[8];
    int M, count;
    while (scanf("%7s %d %d", kind, &M, &count) == 3) {
        if (count < 0 || count > kMostItems) return 1;
        const bool w8 = strcmp(kind, "w8") == 0;
        std::vector<qail_w4a16_item> four(count);
        std::vector<qail_w8a16_item> eight(count);
        for (int i = 0; i < count; ++i) {
            qail_wdesc d;
            memset(&d, 0, sizeof(d));
            if (scanf("%d %d %d", &d.N, &d.K, &d.group_size) != 3) return 1;
            d.scheme = w8 ? QAIL_W8_SYM_GROUP : QAIL_W4_ASYM_GROUP;
            uint32_t* const any = reinterpret_cast<uint32_t*>(0x1000);
            uint16_t* const half = reinterpret_cast<uint16_t*>(0x1000);
            uint16_t* const x = reinterpret_cast<uint16_t*>(kX + i * kApart);
            four[i].d = d; four[i].qweight = any; four[i].scales = half; four[i].zeros = any; four[i].x = x; four[i].y = half;
            eight[i].d = d; eight[i].qweight = any; eight[i].scales = half; eight[i].x = x; eight[i].y = half;
        }
        auto asked = [&](const std::vector<int>& which) {
            std::vector<qail_w4a16_item> f;
            std::vector<qail_w8a16_item> e;
            for (int i : which) {
                f.push_back(four[i]);
                e.push_back(eight[i]);
            }
            size_t b = 0;
            const int st = w8 ? qail_w8a16_batch_workspace_(e.data(), (int)e.size(), M, &b) : qail_w4a16_batch_workspace_(f.data(), (int)f.size(), M, &b);
            return st == QAIL_OK ? b : (size_t)-1;
        };
        std::vector<int> all;
        for (int i = 0; i < count; ++i) all.push_back(i);
        const size_t need = asked(all);
        void* const ws = reinterpret_cast<void*>(1ull << 50);
        launches.clear();
        const int st = w8 ? qail_w8a16_linear_batch_(eight.data(), count, M, ws, need, nullptr)
                          : qail_w4a16_linear_batch_(four.data(), count, M, ws, need, nullptr);
        printf("list %d %zu %zu\n", st, need, launches.size());
        for (const Launch& l : launches) {
            printf("%s %u %zu", l.kernel.c_str(), l.blocks, asked(l.items));
            for (int i : l.items) printf(" %d", i);
            if (!l.variants.empty()) printf(" |");
            for (const auto& v : l.variants) printf(" %d.%d", v.first, v.second);
            printf("\n");
        }
    }
    return 0;
}
