// One call of the library's C interface on the CPU build (see hip/hip_runtime.h):
//   main lx ly lz lt bc_t max_L layout kind kappa csw call prec L j loss in out
// "in" holds the links (4, V, 3, 3), then theta (3, 9, 4, 4) in complex64, then blocks A and B of
// L columns; "out" takes what the call returns.  Inputs and outputs of the call are allocated to
// the byte.
#include <hip/hip_runtime.h>

#include <string>

#include "wdsolve.h"

template <class T>
struct Buf {
    T* p;
    size_t n;
    explicit Buf(size_t n_) : n(n_) { hipMalloc((void**)&p, n * sizeof(T)); }
    ~Buf() { hipFree(p); }
    void read(FILE* f) {
        if (fread(p, sizeof(T), n, f) != n) lanes::fail("short input");
    }
    void write(FILE* f) const { fwrite(p, sizeof(T), n, f); }
};

#define CHECK(e)                                                          \
    do {                                                                  \
        const int r_ = (e);                                               \
        if (r_) {                                                         \
            fprintf(stderr, "%s: %d\n", #e, r_);                          \
            return 3;                                                     \
        }                                                                 \
    } while (0)

int main(int argc, char** argv) {
    if (argc != 18) return 2;
    const int dims[4] = {atoi(argv[1]), atoi(argv[2]), atoi(argv[3]), atoi(argv[4])};
    const size_t V = (size_t)dims[0] * dims[1] * dims[2] * dims[3];
    const int bc = atoi(argv[5]), max_L = atoi(argv[6]), layout = atoi(argv[7]), kind = atoi(argv[8]);
    const double kappa = atof(argv[9]), csw = atof(argv[10]);
    const std::string call = argv[11];
    const int prec = atoi(argv[12]), L = atoi(argv[13]), j = atoi(argv[14]), loss = atoi(argv[15]);
    FILE* in = fopen(argv[16], "rb");
    FILE* out = fopen(argv[17], "wb");
    if (!in || !out) return 2;
    Buf<double> U(4 * 9 * 2 * V), A(24 * V * L), B(24 * V * L), Y(24 * V * L);
    Buf<float> theta(3 * 9 * 16 * 2);
    U.read(in);
    theta.read(in);
    A.read(in);
    B.read(in);
    wd_ctx* c = nullptr;
    CHECK(wd_create(&c, dims, bc, max_L, nullptr));
    CHECK(wd_set_links(c, U.p, j % 2));
    CHECK(wd_set_params(c, kappa, csw, kind));
    CHECK(wd_set_layout(c, layout));
    CHECK(wd_set_learned(c, theta.p));
    if (call == "apply") {
        CHECK(wd_apply(c, A.p, Y.p, L, prec));
        Y.write(out);
    } else if (call == "jacobi") {
        CHECK(jacobi_precond(c, A.p, Y.p, L, j, prec));
        Y.write(out);
    } else if (call == "learned") {
        CHECK(wd_learned_apply(c, A.p, Y.p, L, prec));
        Y.write(out);
    } else if (call == "grad") {
        Buf<double> lv(1), G(3 * 9 * 16 * 2);
        CHECK(wd_learned_grad(c, A.p, B.p, L, loss, lv.p, G.p));
        lv.write(out);
        G.write(out);
    } else if (call == "gram") {
        Buf<double> C(2 * L * L);
        CHECK(wd_block_gram(c, A.p, B.p, L, C.p));
        C.write(out);
        CHECK(wd_block_gram_static(A.p, B.p, 12 * V, L, C.p, nullptr));
        C.write(out);
    } else if (call == "solve" || call == "stab") {
        wd_solve_opts o{};
        o.j = j;
        o.precond = j > 0 ? WD_PRECOND_JACOBI : WD_PRECOND_NONE;
        o.prec_inner = prec;
        o.max_restarts = -1;
        wd_solve_info info{};
        CHECK((call == "solve" ? bbicggr_solve : bbicgstab_solve)(c, A.p, Y.p, L, 1e-10, &o, &info));
        Y.write(out);
    } else {
        return 2;
    }
    CHECK(wd_destroy(c));
    fclose(out);
    fclose(in);
    return 0;
}
