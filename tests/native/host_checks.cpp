// Host logic of the library that no entry point shows without a GPU: plans of architecture descriptions and the request store's
// allocations, with the runtime's allocators replaced.  Built by tests/test_host_logic.py against libcoe.so, with the host code of
// coe.cpp compiled in under the address and undefined-behaviour sanitizers.
//   host_checks plan < descriptions      a description: dtype h w c classes n_layers and 12 words a layer; prints the plan of each
//   host_checks store <max_requests> <max_stages> <classes> <pinned bytes to be had>      prints status, pinned words, message
#include "../../paper_2503_02354_amd/csrc/coe.cpp"

#include <cstdlib>
#include <iostream>

static size_t g_pinned_left = 0;
extern "C" {
hipError_t hipMalloc(void** p, size_t) { *p = std::malloc(1); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned int)
{
    *p = nullptr;
    if (bytes > g_pinned_left) return hipErrorOutOfMemory;
    g_pinned_left -= bytes;
    *p = std::malloc(1);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}

static int plans()
{
    coe_arch_desc d{};
    while (std::cin >> d.dtype >> d.in_h >> d.in_w >> d.in_c >> d.n_classes >> d.n_layers) {
        std::vector<coe_layer> layers(d.n_layers);
        for (coe_layer& l : layers)
            for (int32_t* w : {&l.op, &l.src, &l.dst, &l.res, &l.k, &l.r, &l.s, &l.stride, &l.pad, &l.act, &l.aux0, &l.aux1})
                if (!(std::cin >> *w)) return 1;
        d.layers = layers.data();
        coe_ctx c{};
        ArchPlan a;
        std::cout << "rc " << plan_arch(&c, &d, a);
        for (const LayerPlan& L : a.layers) {
            const bool head = L.d.op == COE_OP_HEAD || L.d.op == COE_OP_HEAD_CLS || L.d.op == COE_OP_HEAD_DET;
            const bool res = L.d.op == COE_OP_CONV || L.d.op == COE_OP_CONCAT || L.d.op == COE_OP_HEAD_DET;
            std::cout << " | " << L.d.op << ' ' << L.src << ' ' << (head ? -1 : L.dst) << ' ' << (res ? L.res : -1) << ' ' << L.fused_away << L.pairs;
            for (int i = 0; i < L.n_sources; ++i) std::cout << " s" << L.source[i];
        }
        for (size_t e : a.buf_elems) std::cout << ' ' << e;
        std::cout << '\n';
    }
    return 0;
}

int main(int argc, char** argv)
{
    if (argc == 2 && std::string(argv[1]) == "plan") return plans();
    if (argc == 6 && std::string(argv[1]) == "store") {
        coe_ctx c{};
        c.cfg.max_requests = std::atoi(argv[2]);
        c.cfg.max_stages = std::atoi(argv[3]);
        c.max_classes = std::atoi(argv[4]);
        g_pinned_left = std::strtoull(argv[5], nullptr, 10);
        ArchPlan a{};
        a.in_h = a.in_w = a.in_c = 1;
        c.archs.push_back(a);
        const int rc = ensure_store(&c);
        std::cout << rc << ' ' << c.out_words << ' ' << (c.h_out != nullptr) << ' ' << c.err << '\n';
        return 0;
    }
    return 2;
}
