// wcnst_gridcheck LIB NX NY ROWS: prints the workgroups of a 2D solver's
// right-hand-side launch with segments of ROWS rows (0: the default), and the
// rows that wcnst_stage_shape reports, over a stand-in for the HIP runtime
// (hip_stand_in.hpp).
#include <dlfcn.h>
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
    SYM(wcnst_set_tuning);
    SYM(wcnst_stage_shape);
    SYM(wcnst_rhs);
    SYM(wcnst_destroy);
    wcnst_desc d;
    if (wcnst_desc_init_(&d)) return 3;
    d.ndim = 2;
    d.nx = atoi(argv[2]);
    d.ny = atoi(argv[3]);
    size_t bytes = 0;
    if (wcnst_workspace_size_(&d, &bytes)) return 3;
    void* ws = cells(bytes);
    double U = 0.0, R = 0.0;  // (no kernel runs)
    wcnst_solver* s = nullptr;
    int strips, rows1, rows2, nseg1, nseg;
    if (wcnst_create_(&d, nullptr, ws, bytes, &s) || wcnst_set_tuning_(s, atoi(argv[4])) || wcnst_rhs_(s, &U, &R, nullptr) ||
        wcnst_stage_shape_(s, &strips, &rows1, &rows2, &nseg1, &nseg))
        return 4;
    printf("%llu %d\n", last_groups, rows1);
    wcnst_destroy_(s);
    free(ws);
    return 0;
}
