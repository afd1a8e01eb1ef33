// Assembly, products, solves and serving of the igaefie library through its C ABI, for sanitizer
// runs against the stand-in runtime (tests/hip_stand_in.cpp): every kind, degree and precision on
// small objects, then servers of three to six workers with single waves, several waves, refined
// solves, merging and small budgets, polled while they run.
//
// usage: serve_driver <geometry file> <servers> (file as for host_driver.cpp)
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../include/igaefie.h"

namespace {

struct GeomData {
    int P = 0;
    std::vector<int> deg, nctrl;
    std::vector<double> knots, ctrl;
};

bool read_geom(const char *path, GeomData &g)
{
    FILE *f = std::fopen(path, "rb");
    if (!f) return false;
    int32_t P = 0;
    int64_t nk = 0, nc = 0;
    bool ok = std::fread(&P, 4, 1, f) == 1 && P > 0 && P < 10000;
    if (ok) {
        g.P = P;
        g.deg.resize(2 * P);
        g.nctrl.resize(2 * P);
        ok = std::fread(g.deg.data(), 4, 2 * P, f) == (size_t)(2 * P) &&
             std::fread(g.nctrl.data(), 4, 2 * P, f) == (size_t)(2 * P) && std::fread(&nk, 8, 1, f) == 1;
    }
    if (ok) {
        g.knots.resize(nk);
        ok = std::fread(g.knots.data(), 8, nk, f) == (size_t)nk && std::fread(&nc, 8, 1, f) == 1;
    }
    if (ok) {
        g.ctrl.resize(4 * nc);
        ok = std::fread(g.ctrl.data(), 8, 4 * nc, f) == (size_t)(4 * nc);
    }
    std::fclose(f);
    return ok;
}

#define CHECK(call)                                                                                      \
    do {                                                                                                 \
        const int rc_ = (call);                                                                          \
        if (rc_ < 0 && rc_ != IGE_ENOTCONV) {                                                            \
            std::fprintf(stderr, "line %d: status %d: %s\n", __LINE__, rc_, ige_last_error());           \
            std::exit(3);                                                                                \
        }                                                                                                \
    } while (0)

void direct(ige_geom geom, int kind, int p, int m)
{
    ige_params P{p, m, 3.0, 4 + p, m == 2 ? 1.0 : 1.6, 4, 4, m > 1 ? 1 : -1, -1, 0.0, kind};
    if (m == 3) {   // a degree per level
        P.q_level[1] = 9;
        P.q_level[2] = 5 + p;
    }
    if (m == 2 && p == 2) P.store_coupling = 1;
    ige_op op = nullptr;
    CHECK(ige_op_assemble(geom, &P, &op));
    ige_op_info_t info{};
    CHECK(ige_op_info(op, &info));
    const size_t N = (size_t)info.n_dof;
    for (int r : {1, 2, 9, 33}) {
        std::vector<ige_c64> x(N * r), y(N * r), pol(3 * r);
        std::vector<double> a(3 * (size_t)r, 0.5);
        if (kind == IGE_OP_SCALAR) CHECK(ige_rhs_scalar(op, r, r & 1, a.data(), x.data(), IGE_HOST));
        else CHECK(ige_rhs_plane_wave(op, r, a.data(), pol.data(), x.data(), IGE_HOST));
        for (int prec = IGE_F64; prec <= IGE_BF16X3_ALL; ++prec) CHECK(ige_apply_prec(op, r, x.data(), y.data(), IGE_HOST, prec));
        ige_solve_opts o{1e-6, 7, 20, 0, 1e-4, IGE_F32};
        std::vector<ige_solve_stats> st(r);
        CHECK(ige_solve(op, r, x.data(), y.data(), IGE_HOST, &o, st.data()));
        for (int ip : {IGE_F64, IGE_F32, IGE_BF16X3_ALL}) {
            o.refine = 1;
            o.inner_prec = ip;
            o.restart = 5;
            CHECK(ige_solve(op, r, x.data(), y.data(), IGE_HOST, &o, st.data()));
        }
        std::vector<double> pts(3 * 17, 3.0);
        std::vector<ige_c64> E(17 * 3 * (size_t)r);
        CHECK(ige_potential(op, r, x.data(), IGE_HOST, 17, pts.data(), E.data()));
        int choice[7];
        if (r > 1) CHECK(ige_op_autotune(op, r, r & 1 ? IGE_F64 : IGE_BF16X3_ALL, choice, 7));
    }
    std::vector<ige_c64> near((size_t)info.near_nnz);
    CHECK(ige_op_near_blocks(op, near.data(), info.near_nnz));
    CHECK(ige_op_destroy(op));
}

void serve(ige_ctx ctx, ige_geom geom, int k)
{
    ige_srv srv = nullptr;
    CHECK(ige_srv_create(ctx, 3 + k % 4, k % 3 ? 0 : (size_t)60 << 20, &srv));
    if (k % 2) CHECK(ige_srv_set_merge(srv, 1 + k % 20));
    std::vector<int64_t> ticket;
    std::vector<int> waves;
    for (int i = 0; i < 14; ++i) {
        ige_params P{1 + i % 3, 1 + i % 3, 2.0 + i % 2, 4 + i % 3, 1.0, 4, 4, 1, 0, 0.0, IGE_OP_EFIE};
        const int w = i % 4 == 1 ? 9 : (i % 4 == 2 ? 3 : 1);
        std::vector<double> d(3 * (size_t)w, 0.5);
        std::vector<ige_c64> pol(3 * (size_t)w);
        ige_solve_opts o{1e-6, 20, 40, i % 3 == 0, 1e-4, i % 3 == 0 ? IGE_BF16X3_ALL : IGE_F64};
        int64_t t = 0;
        const int rc = ige_srv_submit_waves(srv, geom, &P, w, d.data(), pol.data(), &o, &t);
        if (rc == IGE_ENOMEM) continue;   // beyond the small budget
        CHECK(rc);
        ticket.push_back(t);
        waves.push_back(w);
    }
    for (size_t i = 0; i < ticket.size(); ++i) {
        ige_srv_stats st{};
        do {
            CHECK(ige_srv_poll(srv, ticket[i], &st));
        } while (st.state != 2);
        CHECK(ige_srv_wait(srv, ticket[i], &st));
        CHECK(st.rc);
        std::vector<ige_c64> x((size_t)st.n_dof * waves[i]);
        CHECK(ige_srv_result(srv, ticket[i], x.data(), (int64_t)x.size()));
    }
    CHECK(ige_srv_destroy(srv));
}

}  // namespace

int main(int argc, char **argv)
{
    GeomData gd;
    if (argc < 3 || !read_geom(argv[1], gd)) {
        std::fprintf(stderr, "usage: %s <geometry file> <servers>\n", argv[0]);
        return 2;
    }
    ige_ctx ctx = nullptr;
    ige_geom geom = nullptr;
    CHECK(ige_ctx_create(0, nullptr, &ctx));
    CHECK(ige_geom_create(ctx, gd.P, gd.deg.data(), gd.nctrl.data(), gd.knots.data(), gd.ctrl.data(), &geom));
    for (int kind : {IGE_OP_EFIE, IGE_OP_SCALAR})
        for (int p = 1; p <= 4; ++p)
            for (int m = 1; m <= 3; ++m)
                if (p < 4 || m < 3) direct(geom, kind, p, m);
    for (int k = 0; k < std::atoi(argv[2]); ++k) serve(ctx, geom, k);
    CHECK(ige_geom_destroy(geom));
    CHECK(ige_ctx_destroy(ctx));
    std::printf("serve driver: all done\n");
    return 0;
}
