/* launch_rule.cpp -- what the library would launch, on the host alone.
 *
 * The library's host source compiled into a program whose HIP entry points record
 * instead of queueing, so that the launch rule can be read for any grid without a
 * GPU (compiled for the host only: no device code).  One request per line of
 * standard input:
 *     call op bc_mode ndim n0 [n1 [n2 [n3]]]
 * with call one of fwd, fwdR (residuals stored), fwd_ws, bwd, vg, vg_ws, bc, vjp, vjp_acc.
 * One answer per launch,
 *     <device kernel name> <workgroups> <threads> [<chunk length> <tiles_x> <tiles_y>]
 * (the bracket for the marching kernels), then "= <status>".  With the argument
 * "kernels": the names of the library's kernels instead; with "residency": what the rule
 * takes for the workgroups of each tile per CU, one line per tile,
 *     <fwd|fwdR|bwd|vg|vjp> <op> <tile width> <height> <not periodic> <periodic>
 */
#include "fpde.hip"

#include <stdio.h>
#include <string.h>

#include <map>
#include <string>

static std::map<const void*, std::string> g_names;

extern "C" {
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
    g_names[host] = name;
}
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t, hipStream_t) {
    const std::string& name = g_names[f];
    printf("%s %u %u", name.c_str(), grid.x, block.x);
    if (name.find("4Dims") != std::string::npos) {  // (Ptrs, Dims, ...)
        const fpde::Dims& d = *(const fpde::Dims*)args[1];
        printf(" %d %d %d", d.zc, d.tiles_x, d.tiles_y);
    }
    printf("\n");
    return hipSuccess;
}
}

template <class T>
static void show_tile(const char* kind, int op, bool loss) {
    printf("%s %d %d %d %d %d\n", kind, op, T::TX, T::TY, T::res(loss, false), T::res(loss, true));
}
template <class P>
static void show(const char* kind, int op, const P&, bool loss) {
    show_tile<typename P::W>(kind, op, loss);
    show_tile<typename P::N>(kind, op, loss);
}
static void show_residency() {
    for (int op = FPDE_BURGERS_1DT; op <= FPDE_NS_3DT; ++op)
        fpde::with_op(op, [&](auto tag) {
            using GEO = typename decltype(tag)::GEO;
            show("fwd", op, GEO::FWD, true);
            show("fwdR", op, GEO::FWDR, true);
            show("vjp", op, GEO::VJP, false);
            if constexpr (!decltype(tag)::OP::TIME) {  // (the time march: one per CU)
                show("bwd", op, GEO::BWD, false);
                show("vg", op, GEO::VG, true);
                if constexpr (!GEO::D3) show("vg", op, GEO::VGA, true);
            }
            return FPDE_OK;
        });
}

int main(int argc, char** argv) {
    if (argc > 1) {
        if (!strcmp(argv[1], "residency")) show_residency();
        else
            for (const auto& k : g_names) printf("%s\n", k.second.c_str());
        return 0;
    }
    // device addresses far apart, never dereferenced
    const float *f[4], *c[6], *s[4];
    float* o[4];
    for (uintptr_t i = 0; i < 6; ++i) c[i] = (const float*)((i + 10) << 44);
    for (uintptr_t i = 0; i < 4; ++i) {
        f[i] = (const float*)((i + 1) << 44);
        s[i] = (const float*)((i + 20) << 44);
        o[i] = (float*)((i + 30) << 44);
    }
    double *loss = (double*)(40ull << 44), *dl = (double*)(41ull << 44);
    void* ws = (void*)(42ull << 44);
    const fpde_coeffs co = {0.01, 1.0, 0.1, 0.1};
    char call[16];
    int op, bc, nd;
    while (scanf("%15s %d %d %d", call, &op, &bc, &nd) == 4) {
        fpde_grid4 g = {};
        g.ndim = nd;
        g.bc_mode = bc;
        for (int a = 0; a < nd; ++a) {
            long long n;
            if (scanf("%lld", &n) != 1) return 1;
            g.n[a] = n;
            g.h[a] = 0.1;
        }
        int st = -100;
        const std::string w = call;
        if (w == "fwd") st = fpde_residual_fwd4(op, &g, &co, f, c, nullptr, loss, nullptr);
        if (w == "fwdR") st = fpde_residual_fwd4(op, &g, &co, f, c, o, loss, nullptr);
        if (w == "fwd_ws") st = fpde_residual_fwd_ws4(op, &g, &co, f, c, nullptr, loss, ws, nullptr);
        if (w == "bwd") st = fpde_residual_bwd4(op, &g, &co, f, c, dl, o, nullptr);
        if (w == "bc") st = fpde_bc_correct4(op, &g, &co, f, c, dl, o, nullptr);
        if (w == "vjp") st = fpde_residual_vjp4(op, &g, &co, f, s, 0, o, nullptr);
        if (w == "vjp_acc") st = fpde_residual_vjp4(op, &g, &co, f, s, 1, o, nullptr);
        if (w == "vg")
            st = fpde_residual_value_and_grad4(op, &g, &co, f, c, dl, loss, o, nullptr);
        if (w == "vg_ws")
            st = fpde_residual_value_and_grad_ws4(op, &g, &co, f, c, dl, loss, o, ws, nullptr);
        printf("= %d\n", st);
    }
    return 0;
}
