// Host logic of the library that no entry point shows without a GPU: plans of architecture descriptions.  Built by
// tests/test_host_logic.py against libcoe.so, with the host code of coe.cpp compiled in under the address and undefined-behaviour
// sanitizers.
//   host_checks plan < descriptions      a description: dtype h w c classes n_layers and 12 words a layer; prints the plan of each
#include "../../paper_2503_02354_amd/csrc/coe.cpp"

#include <iostream>

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
    return 2;
}
