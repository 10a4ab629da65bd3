// CPU run of the kernels with one wave or one block per cell through the host stand-in for the HIP runtime
// (hip/hip_runtime.h beside this file), for the sanitizer test.  Test infrastructure.
//
//   emu_cells <mechanism file> <form> <input> <output>
//     form:   "queue"  one wave per cell, cells claimed from an order (last cell first)
//             "plain"  one wave per cell, without an order
//             "list"   one wave per cell, every second cell through a list with its length in memory
//             "tape"   one wave per cell with a tape and a queue, then the reverse sweep with seeds of one
//             "block"  one block of eight waves per cell
//     input:  int64 n; double dt; double p[n], T[n], Y[K][n]
//     output: double T[n], Y[K][n]; int32 status[n], n_steps[2n]; for "tape" double T0_bar[n], Y0_bar[K][n], lnA_bar[M][n]
#include <cstdio>
#include <cstring>
#include <vector>

#include "df_internal.h"

int main(int argc, char **argv) {
    if (argc != 5) return 2;
    df_mech *m = nullptr;
    if (df_mech_load(argv[1], 0, &m) != DF_OK) {
        std::fprintf(stderr, "df_mech_load: %s\n", df_last_error());
        return 1;
    }
    const int K = m->host.K, M = m->host.M;
    FILE *f = std::fopen(argv[3], "rb");
    if (!f) return 1;
    int64_t n = 0;
    double dt = 0.0;
    bool ok = std::fread(&n, 8, 1, f) == 1 && std::fread(&dt, 8, 1, f) == 1 && n > 0;
    std::vector<double> p(n), T(n), Y(size_t(K) * n), rr(size_t(K) * n);
    ok = ok && std::fread(p.data(), 8, n, f) == size_t(n) && std::fread(T.data(), 8, n, f) == size_t(n) &&
         std::fread(Y.data(), 8, Y.size(), f) == Y.size();
    std::fclose(f);
    if (!ok) return 1;
    std::vector<int32_t> st(n, -7), ns(2 * n, -7), order(n);
    df_chem_opts o;
    df_chem_default_opts(&o);
    df::StepArgs a{n, n, dt, nullptr, p.data(), T.data(), Y.data(), nullptr, rr.data(), st.data(), ns.data(),
                   df::kernel_opts(o), DF_CELL_OK};
    std::vector<unsigned long long> ctr(size_t(df::kCellQueues) * 16, 0);
    const std::string form(argv[2]);
    constexpr int kCap = 256;
    std::vector<double> tape, out;
    df_status r = DF_OK;
    if (form == "block") {
        r = df::chem_block_supported(m->dev) ? df::launch_chem_block(m->dev, a, nullptr, nullptr, nullptr) : DF_E_UNSUPPORTED;
    } else if (form == "list") {
        int32_t count = 0;
        for (int64_t i = 0; i < n; i += 2) order[count++] = int32_t(i);
        for (int64_t i = 1; i < n; i += 2) st[i] = 0, ns[i] = ns[n + i] = 0;
        r = df::launch_chem_cell(m->dev, a, df::CellQueue{order.data(), &count, nullptr, nullptr, nullptr, 0}, nullptr);
    } else if (form == "plain") {
        r = df::launch_chem_cell(m->dev, a, df::CellQueue{nullptr, nullptr, nullptr, nullptr, nullptr, 0}, nullptr);
    } else {
        for (int64_t i = 0; i < n; ++i) order[i] = int32_t(n - 1 - i);
        if (form == "tape") {
            a.rr = nullptr;
            tape.assign(df::tape_bytes(K, n, kCap) / 8, 0.0);
            a.tape = tape.data();
            a.tape_cap = kCap;
        }
        r = df::launch_chem_cell(m->dev, a, df::CellQueue{nullptr, nullptr, order.data(), ctr.data(), nullptr, 0}, nullptr);
        if (r == DF_OK && form == "tape") {
            const std::vector<double> Tb(n, 1.0), Yb(size_t(K) * n, 1.0);
            std::vector<double> wth(size_t(M) * n);
            out.assign(size_t(1 + K + M) * n, -7.0);
            r = df::launch_sweep_cell(m->dev, n, n, p.data(), tape.data(), kCap, Tb.data(), Yb.data(), out.data(),
                                      out.data() + n, out.data() + size_t(1 + K) * n, wth.data(), nullptr, nullptr);
        }
    }
    if (r != DF_OK) {
        std::fprintf(stderr, "step: %s\n", df_last_error());
        return 1;
    }
    f = std::fopen(argv[4], "wb");
    if (!f) return 1;
    std::fwrite(T.data(), 8, n, f);
    std::fwrite(Y.data(), 8, Y.size(), f);
    std::fwrite(st.data(), 4, n, f);
    std::fwrite(ns.data(), 4, 2 * n, f);
    if (!out.empty()) std::fwrite(out.data(), 8, out.size(), f);
    std::fclose(f);
    df_mech_free(m);
    return 0;
}
