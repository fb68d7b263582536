// Plays passes of the minimizer on the CPU: prints one line per check,
// "name ok" or "name FAILED ...".
#include "ff_optim.hip"

using namespace ff;
using hostsim::Group;

namespace {

// One system of 20 atoms whose accept pass has `bx` workgroups in each of
// `rows` product rows.
struct Fixture {
    std::vector<uint64_t> mem;
    Args a{};
    SysInfo* si;
    Ctl* c;
    BatchState* batch;

    Fixture(int bx, int rows) {
        Layout& L = a.L;
        size_t off = 0;
        auto take = [&](size_t b) { const size_t o = off; off += (b + 255) & ~(size_t)255; return o; };
        L.n_sys = 1;
        L.acc_rows = rows;
        L.vstride = 3 * 64;
        L.off_sys = take(sizeof(SysInfo));
        L.off_batch = take(sizeof(BatchState));
        L.off_ctl = take(sizeof(Ctl));
        L.off_map_acc = take(bx * sizeof(int2));
        L.off_red = take((size_t)6 * bx * rows * 8);
        L.off_vec = take((size_t)V_COUNT * L.vstride * 8);
        mem.assign(off / 8, 0);
        a.ws = (char*)mem.data();
        si = sys_info(a);
        si->n = 20;
        si->np = 64;
        si->acc_bx = bx;
        c = ctl_at(a, 0);
        batch = at<BatchState>(a.ws, L.off_batch);
        for (int b = 0; b < bx; ++b) at<int2>(a.ws, L.off_map_acc)[b] = int2{0, b};
    }
    // A control block as ff_minimize starts it.
    void kick(int method) {
        MinParamsDev p{};
        p.method = method;
        p.max_iter = 100;
        p.tol = 1e-3;
        p.h_init = 0.1;
        p.ls_K = 2;
        p.precision = P_FP64;
        Group g([&] { k_kick(a, p, 0, nullptr, 0); }, dim3(0), dim3(1), 256);
        g.finish();
    }
    // ... and as the first accepted step leaves it for the accept pass.
    void accept() {
        c->e[0] = 2.0; c->e[1] = 1.0;
        c->g2[0] = c->g2[1] = 1.0;
        c->ginf[0] = c->ginf[1] = 1.0;
        c->accept = 1;
        c->acc_new = 1;
        c->acc_old = 0;
        c->acc_rows = 0;
        c->best = 0;
        c->action = ACT_NONE;
    }
};

void result(const char* name, bool ok, const char* why) { std::printf("%s %s\n", name, ok ? "ok" : why); }

// Workgroups without a product row: whatever the order in which their
// wavefronts start, all wavefronts of a workgroup take part in the pass and
// its last workgroup makes the decision once.
void accept_order(const char* name, int method, int bx, int rows) {
    Fixture f(bx, rows);
    f.kick(method);
    f.accept();
    const int n = bx * rows;
    auto kernel = [&] { k_accept(f.a); };
    // every workgroup but the last: the first wavefront as far as it gets, the
    // others not yet started
    std::vector<std::unique_ptr<Group>> groups;
    for (int k = 0; k < n; ++k)
        groups.emplace_back(new Group(kernel, dim3(k % bx, k / bx), dim3(bx, rows), kFinBlock));
    for (int k = 0; k < n - 1; ++k) groups[k]->run(0, 64);
    groups[n - 1]->finish();
    bool divergent = false;
    for (int k = 0; k < n; ++k) {
        groups[k]->finish();
        divergent |= groups[k]->divergent;
    }
    result(name, !divergent, "FAILED: part of a workgroup left the pass while its siblings wait at a barrier");
    result(name, f.c->iters == 1 && f.c->accept == 0 && f.c->action == ACT_EVAL && f.c->acc_ticket == 0,
           "FAILED: not one decision");
}

// Counts that something left behind do not outlive the start of a minimization.
void kick_counts(const char* name, int resume) {
    Fixture f(1, 2);
    f.kick(M_GD);
    f.accept();
    f.c->fin_ticket = 3;
    f.c->acc_ticket = 1;
    MinParamsDev p = f.c->p;
    Group g([&] { k_kick(f.a, p, resume, nullptr, 0); }, dim3(0), dim3(1), kFinBlock);
    g.finish();
    result(name, f.c->fin_ticket == 0 && f.c->acc_ticket == 0, "FAILED: counts are kept");
}

}  // namespace

int main() {
    accept_order("accept_gd", M_GD, 1, 2);
    accept_order("accept_hb", M_HB, 1, 11);
    accept_order("accept_fgm", M_FGM, 3, 5);
    kick_counts("kick_counts", 0);
    kick_counts("resume_counts", 1);
    return 0;
}
