// Tile-shape autotuner.
#include <chrono>
#include <cmath>
#include <cstring>
#include <thread>
#include <vector>

#include "cp_internal.h"

namespace cp {

namespace {

// Deterministic synthetic charge for timing: a hash of the node index mapped
// to [-1, 1] x 1e-4 C/m^3 (only the launch shapes are being timed).
__global__ void k_fill_hash(double* x, long long n) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    unsigned long long h = (unsigned long long)i * 0x9E3779B97F4A7C15ull;
    h ^= h >> 31;
    h *= 0xBF58476D1CE4E5B9ull;
    h ^= h >> 29;
    x[i] = ((double)(h >> 11) * (1.0 / 9007199254740992.0) * 2.0 - 1.0) * 1e-4;
}

struct Candidate {
    const char* key;
    std::vector<double> values;
};

}  // namespace

}  // namespace cp

using namespace cp;

extern "C" {

int cylpoisson_autotune(cylpoisson_plan* p, void* stream) {
    if (!p) {
        set_error("plan must not be NULL");
        return CYLPOISSON_EINVAL;
    }
    int prev_dev = 0;
    (void)hipGetDevice(&prev_dev);
    (void)hipSetDevice(p->device);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const long long n = (long long)p->nt * p->nz * p->nr;
    double* rho = nullptr;
    double* phi = nullptr;
    int status = CYLPOISSON_OK;
    if (hipMalloc(&rho, n * sizeof(double)) != hipSuccess || hipMalloc(&phi, n * sizeof(double)) != hipSuccess) {
        (void)hipGetLastError();
        if (rho) (void)hipFree(rho);
        (void)hipSetDevice(prev_dev);
        set_error("autotune: cannot allocate two node arrays");
        return CYLPOISSON_ENOMEM;
    }
    k_fill_hash<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(rho, n);
    const Options saved = p->opt;
    // a fixed amount of work per trial: two cycles, never converged
    p->opt.max_cycles = 2;
    p->opt.timing = 0;
    p->opt.warm_start = 0;
    auto trial = [&](double* ms) -> int {
        drop_graphs(p);
        for (int rep = 0; rep < 4; ++rep) {
            const auto t0 = std::chrono::steady_clock::now();
            const int st = cylpoisson_solve(p, rho, phi, 1e-300, stream);
            if (st != CYLPOISSON_OK && st != CYLPOISSON_NOT_CONVERGED) return st;
            if (hipStreamSynchronize(s) != hipSuccess) return CYLPOISSON_EHIP;
            const double t = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
            if (rep == 1 || (rep > 1 && t < *ms)) *ms = t;  // first run warms up
        }
        return CYLPOISSON_OK;
    };
    const int rows = p->nz - 2;
    std::vector<Candidate> cands = {
        {"chunk_rows", {0, 32, 48, 64, 96, 128, 192, 256}},
        {"chunk_rows_coarse", {0, 16, 24, 32, 48, 64}},
        {"groups", {1, 2, 4}},
    };
    double best = INFINITY;
    status = trial(&best);
    for (const Candidate& c : cands) {
        double keep = 0.0;
        (void)cylpoisson_plan_get_option(p, c.key, &keep);
        for (double v : c.values) {
            if (v == keep) continue;
            if ((!std::strcmp(c.key, "chunk_rows") || !std::strcmp(c.key, "chunk_rows_coarse")) && v > rows)
                continue;
            if (cylpoisson_plan_set_option(p, c.key, v) != CYLPOISSON_OK) continue;
            double t = INFINITY;
            const int st = trial(&t);
            if (st != CYLPOISSON_OK) {
                status = st;
                break;
            }
            if (t < 0.97 * best) {  // keep a change only for a clear gain
                best = t;
                keep = v;
            }
        }
        (void)cylpoisson_plan_set_option(p, c.key, keep);
        if (status != CYLPOISSON_OK) break;
    }
    // The relaxation factor (option tune_omega, point smoother V-cycles only):
    // the contraction per cycle from cycle 2 to cycle 6 of a solve from zero
    // on the same charge (the check after a solve's last cycle is always
    // formed), for each candidate; omega changes only for a clear gain.
    double omega = saved.omega;
    if (status == CYLPOISSON_OK && saved.tune_omega && saved.smoother == 0 && saved.krylov == 0) {
        p->opt.fmg = 0;
        auto contraction = [&](double w, double* rate) -> int {
            p->opt.omega = w;
            double rel[2] = {0.0, 0.0};
            int cyc[2] = {0, 0};
            const int maxc[2] = {2, 6};
            for (int i = 0; i < 2; ++i) {
                p->opt.max_cycles = maxc[i];
                drop_graphs(p);
                const int st = cylpoisson_solve(p, rho, phi, 1e-300, stream);
                if (st != CYLPOISSON_OK && st != CYLPOISSON_NOT_CONVERGED) return st;
                rel[i] = p->stats.rel_residual;
                cyc[i] = p->stats.cycles;
            }
            *rate = (cyc[1] > cyc[0] && rel[0] > 0.0 && rel[1] > 0.0)
                        ? std::pow(rel[1] / rel[0], 1.0 / (cyc[1] - cyc[0]))
                        : 1.0;
            return CYLPOISSON_OK;
        };
        double keep_rate = 1.0;
        status = contraction(saved.omega, &keep_rate);
        double best_rate = keep_rate;
        for (double w : {1.0, 1.1, 1.15, 1.2, 1.25, 1.3, 1.35, 1.4, 1.5}) {
            if (status != CYLPOISSON_OK || w == saved.omega) continue;
            double r = 1.0;
            status = contraction(w, &r);
            if (status == CYLPOISSON_OK && r < best_rate) {
                best_rate = r;
                omega = w;
            }
        }
        if (!(best_rate < 0.9 * keep_rate)) omega = saved.omega;
    }
    const Options tuned = p->opt;
    p->opt = saved;
    p->opt.chunk_rows = tuned.chunk_rows;
    p->opt.chunk_rows_coarse = tuned.chunk_rows_coarse;
    p->opt.groups = tuned.groups;
    if (status == CYLPOISSON_OK) p->opt.omega = omega;
    drop_graphs(p);
    (void)hipFree(rho);
    (void)hipFree(phi);
    (void)hipSetDevice(prev_dev);
    return status;
}

}  // extern "C"
