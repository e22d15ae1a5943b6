// The launches of one join, build or probe, without a GPU: the library's engine
// and kernel objects linked against the HIP entry points below, which record a
// launch instead of making it.  Driven by tests/test_launch_plan.py.
//
//   launch_plan <join|build|probe> algo passes b1 b2 tile lds_cap flags n_r n_s
//
// prints the workspace (and table) bytes, then one line per launch: the kernel,
// its workgroups and threads, and what the checks read of its arguments.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../../paper_1307_1955_amd/csrc/engine.h"
#include "../../paper_1307_1955_amd/csrc/hj_side.h"

namespace {

std::map<const void*, std::string>& kernels() {
    static std::map<const void*, std::string> m;
    return m;
}

struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
};
std::vector<Config> pushed;

template <typename T>
const T& arg(void** args, int i) {
    return *static_cast<const T*>(args[i]);
}

}  // namespace

extern "C" {

void** __hipRegisterFatBinary(const void*) {
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    kernels()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
    pushed.push_back(Config{grid, block, lds, stream});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
    const Config c = pushed.back();
    pushed.pop_back();
    *grid = c.grid;
    *block = c.block;
    *lds = c.lds;
    *stream = c.stream;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "none"; }

hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t) {
    const std::string& name = kernels()[fn];
    // (the mangled name holds the kernel's own between its length and the template arguments)
    const size_t k = name.find("k_");
    std::string own;
    for (size_t i = k; i < name.size() && (islower(name[i]) || isdigit(name[i]) || name[i] == '_'); ++i) own += name[i];
    printf("%s grid=%u block=%u lds=%zu", own.c_str(), grid.x, block.x, lds);
    auto ctl = [](const char* what, const hj::ScanCtl& c) { printf(" %s=%u/%u", what, c.max_polls, c.stall); };
    if (own == "k_part_starts") {
        ctl("scan", arg<hj::StartArgs>(args, 1).ctl);
    } else if (own == "k_part_scatter") {
        const hj::SideJob& side = arg<hj::SideJob>(args, 13);
        if (side.kind == hj::kSidePlan) ctl("plan", side.plan.ctl);
        if (arg<hj::ClearTables>(args, 12).table) printf(" clears");
    }
    printf("\n");
    return hipSuccess;
}

}  // extern "C"

namespace hj {
void Recorder::before(const char*) {}
void Recorder::after() { ++n; }
}  // namespace hj

int main(int argc, char** argv) {
    if (argc != 11) return 2;
    const std::string mode = argv[1];
    auto num = [&](int i) { return (uint64_t)strtoull(argv[i], nullptr, 10); };
    hj_params p{};
    p.algo = (uint32_t)num(2);
    p.passes = (uint32_t)num(3);
    p.bits[0] = (uint32_t)num(4);
    p.bits[1] = (uint32_t)num(5);
    p.tile = (uint32_t)num(6);
    p.lds_cap = (uint32_t)num(7);
    p.flags = (uint32_t)num(8);
    const uint64_t n_r = num(9), n_s = num(10);
    // addresses are never read: the launches are only recorded
    char* const base = reinterpret_cast<char*>(uintptr_t{1} << 40);
    int32_t* const col = reinterpret_cast<int32_t*>(uintptr_t{1} << 44);
    const hj_rel R{col, col, n_r}, S{col, col, n_s};
    const hj_out out{col, col, n_s};
    hj::eng::Plan pl;
    if (hj::eng::check_params(&p, n_r, mode == "join" ? n_s : 0, &pl) != HJ_OK) {
        printf("refused: %s\n", hj::eng::last_error());
        return 0;
    }
    hj::Recorder rec;
    hj::eng::init_recorder(rec, nullptr, reinterpret_cast<uint64_t*>(base), true);
    uint64_t* const count = reinterpret_cast<uint64_t*>(col);
    if (mode == "join") {
        printf("bytes %zu\n", hj::eng::ws_bytes_for(pl, n_r, n_s));
        hj::eng::run_join(pl, R, S, out, base, count, rec);
        return 0;
    }
    const size_t table = hj::eng::table_bytes_for(pl, n_r);
    printf("bytes %zu\n", table);
    if (mode == "build") {
        hj::eng::run_build(pl, R, base, rec);
        return 0;
    }
    const hj_table t{pl.res, n_r, col, col, base, table};
    hj::eng::Plan pp;
    if (hj::eng::table_plan(&t, n_s, &pp) != HJ_OK) {
        printf("refused: %s\n", hj::eng::last_error());
        return 0;
    }
    printf("probe bytes %zu\n", hj::eng::probe_bytes_for(pp, n_r, n_s));
    hj::eng::run_probe(pp, t, S, out, base + table, count, rec);
    return 0;
}
