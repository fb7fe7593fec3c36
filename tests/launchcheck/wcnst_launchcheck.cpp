// Whether an entry point reports a kernel launch that fails, over a stand-in
// for the HIP runtime (hip_stand_in.hpp).
//
// wcnst_launchcheck LIB ENTRY NDIM NX: for n = 1, 2, ... prints the status of
// the entry point when its n-th launch fails, then that of a call without a
// failure (for an n beyond its launches), on a line.
#include <dlfcn.h>
#include <math.h>
#include <stdio.h>

#include "hip_stand_in.hpp"

#define SYM(name) auto* name##_ = reinterpret_cast<decltype(&name)>(dlsym(so, #name))

int main(int argc, char** argv)
{
    void* so = argc == 5 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (!so) return 2;
    SYM(wcnst_desc_init);
    SYM(wcnst_workspace_size);
    SYM(wcnst_create);
    SYM(wcnst_step);
    SYM(wcnst_solve);
    SYM(wcnst_solve_noalloc);
    SYM(wcnst_rhs);
    SYM(wcnst_destroy);
    const char* entry = argv[2];
    wcnst_desc d;
    if (wcnst_desc_init_(&d)) return 3;
    d.ndim = atoi(argv[3]);
    d.nx = atoi(argv[4]);
    d.ny = d.ndim == 2 ? d.nx : 1;
    size_t bytes = 0;
    if (wcnst_workspace_size_(&d, &bytes)) return 3;
    const size_t n = sizeof(double) * 4 * (size_t)d.nx * (size_t)d.ny;
    void* ws = cells(bytes);
    double *U = (double*)cells(n), *R = (double*)cells(n);
    for (int k = 1;; ++k) {
        wcnst_solver* s = nullptr;
        fail_at = 0;
        if (wcnst_create_(&d, nullptr, ws, bytes, &s)) return 4;
        launches = 0;
        fail_at = k;
        int st = -1;
        if (!strcmp(entry, "step")) st = wcnst_step_(s, U, 0.0, 0.5);
        if (!strcmp(entry, "step_dt")) st = wcnst_step_(s, U, 0.1, 0.0);
        if (!strcmp(entry, "rhs")) st = wcnst_rhs_(s, U, R, nullptr);
        if (!strcmp(entry, "solve")) st = wcnst_solve_(s, U, INFINITY, 0.5, 3, nullptr, nullptr);
        if (!strcmp(entry, "noalloc"))
            st = wcnst_solve_noalloc_(&d, nullptr, U, INFINITY, 0.5, 3, nullptr, nullptr);
        printf("%d%s", st, k <= launches ? " " : "\n");
        last = hipSuccess;
        wcnst_destroy_(s);
        if (k > launches) return 0;
    }
}
