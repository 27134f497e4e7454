// Which passes lbm_step launches (test code only, on the null device of
// tests/sanitize/null_device.cpp: launches are counted, not executed, and no device memory
// is touched, so domains of any size are cheap).
//
// Input lines: count nx ny bc_x bc_y medium half heat j_plane every mode t n
//   count 1: a single domain; above: a batch of count equal domains
//   mode 0: the default passes; above: lbm_set_time_blocking(mode); below: the same with
//   -mode, a step, and lbm_default_passes
//   t: steps taken before; n: the call
// Output per line: the passes of lbm_step(n), kind and cycles each, as lbm_next_pass
// reports them, "?" after one whose launch was of another kind.
//
// With the argument "reverse" input lines: nx ny bx by medium heat every steps theta. Output:
// the launches of deep, rolling and tile passes that recompute in lbm_backward (theta: with
// parameter gradients), of deep and other adjoint passes, and of deep and other passes of
// lbm_tangent.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "lbm.h"

extern "C" long null_device_launches(const char *sub);

struct Counts {
    long deep, roll, strip, step;
    static Counts now() {
        return Counts{null_device_launches("k_step_deep"), null_device_launches("k_step3_roll"),
                      null_device_launches("k_step4_strip"), null_device_launches("k_step")};
    }
};

static void die(const char *what) {
    std::fprintf(stderr, "%s: %s\n", what, lbm_last_error());
    std::exit(2);
}

static int reverse() {
    int nx, ny, bx, by, medium, heat, every, theta;
    long T;
    while (std::scanf("%d %d %d %d %d %d %d %ld %d", &nx, &ny, &bx, &by, &medium, &heat, &every, &T, &theta) == 9) {
        lbm_desc d;
        lbm_desc_defaults(&d);
        d.nx = nx; d.ny = ny; d.bc_x = bx; d.bc_y = by; d.nu = 0.1; d.dp = 1.0; d.medium = medium; d.ckpt_every = every;
        if (heat) {
            d.thermal.enabled = 1; d.thermal.tau_T = 0.8; d.thermal.Th = 2.0; d.thermal.Tc = 1.0; d.thermal.T0 = 1.5;
        }
        std::vector<float> plane((size_t)nx * ny, 0.5f), out(2 * (size_t)nx * ny);
        size_t bytes = 0;
        if (lbm_workspace_size(&d, T, &bytes) != LBM_OK) die("workspace size");
        void *ws = std::aligned_alloc(4096, (bytes + 4095) / 4096 * 4096);
        lbm_ctx *c = nullptr;
        if (!ws || lbm_create(&d, plane.data(), plane.data(), ws, bytes, nullptr, &c) != LBM_OK) die("create");
        if (lbm_step(c, T) != LBM_OK) die("step");
        const Counts a = Counts::now();
        const long ad = null_device_launches("k_adjoint_deep"), as = null_device_launches("k_adjoint_step");
        double th[4];
        const int rc = theta ? lbm_backward_params(c, out.data(), plane.data(), nullptr, th)
                             : lbm_backward(c, out.data(), plane.data(), nullptr);
        if (rc != LBM_OK) die("backward");
        const Counts b = Counts::now();
        std::printf("%ld %ld %ld %ld %ld", b.deep - a.deep, b.roll - a.roll,
                    (b.step - a.step) - (b.deep - a.deep) - (b.roll - a.roll), null_device_launches("k_adjoint_deep") - ad,
                    null_device_launches("k_adjoint_step") - as);
        const long td = null_device_launches("k_tangent_deep"), ts = null_device_launches("k_tangent_step");
        if (!heat && lbm_tangent(c, plane.data(), nullptr, out.data()) != LBM_OK) die("tangent");
        std::printf(" %ld %ld\n", null_device_launches("k_tangent_deep") - td, null_device_launches("k_tangent_step") - ts);
        lbm_destroy(c);
        std::free(ws);
    }
    return 0;
}

int main(int argc, char **argv) {
    if (argc > 1 && std::strcmp(argv[1], "reverse") == 0) return reverse();
    int count, nx, ny, bx, by, medium, half, heat, j, every, mode;
    long t, n;
    while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %ld %ld", &count, &nx, &ny, &bx, &by, &medium, &half, &heat, &j,
                      &every, &mode, &t, &n) == 13) {
        lbm_desc d;
        lbm_desc_defaults(&d);
        d.nx = nx; d.ny = ny; d.bc_x = bx; d.bc_y = by; d.nu = 0.1; d.dp = 1.0;
        d.medium = medium; d.storage = half ? LBM_FP16_DEV : LBM_FP32_DEV; d.j_plane = j; d.ckpt_every = every;
        if (heat) {
            d.thermal.enabled = 1; d.thermal.tau_T = 0.8; d.thermal.Th = 2.0; d.thermal.Tc = 1.0; d.thermal.T0 = 1.5;
        }
        std::vector<lbm_desc> ds((size_t)count, d);
        std::vector<float> plane(medium == LBM_MEDIUM_UNIFORM ? 0 : (size_t)nx * ny, 0.5f);
        std::vector<const float *> planes((size_t)count, plane.data());
        size_t bytes = 0;
        if ((count > 1 ? lbm_batch_workspace_size(count, ds.data(), &bytes) : lbm_workspace_size(&d, t + n, &bytes)) != LBM_OK)
            die("workspace size");
        void *ws = std::aligned_alloc(4096, (bytes + 4095) / 4096 * 4096);
        lbm_ctx *c = nullptr;
        const int rc = count > 1 ? lbm_create_batch(count, ds.data(), planes.data(), planes.data(), ws, bytes, nullptr, nullptr, &c)
                                 : lbm_create(&d, plane.data(), plane.data(), ws, bytes, nullptr, &c);
        if (!ws || rc != LBM_OK) die("create");
        if (count > 1 && lbm_set_graph_steps(c, 0) != LBM_OK) die("graph steps");
        if (mode && lbm_set_time_blocking(c, std::abs(mode)) != LBM_OK) die("mode");
        if (mode < 0 && (lbm_step(c, 1) != LBM_OK || lbm_default_passes(c) != LBM_OK)) die("default passes");
        if (lbm_step(c, t) != LBM_OK) die("step");
        while (n > 0) {
            int32_t kind = -1, cycles = 0;
            if (lbm_next_pass(c, n, &kind, &cycles) != LBM_OK || cycles < 1 || cycles > n) die("next pass");
            const Counts a = Counts::now();
            if (lbm_step(c, cycles) != LBM_OK) die("step");
            const Counts b = Counts::now();
            const bool deep = b.deep > a.deep, roll = b.roll > a.roll, strip = b.strip > a.strip;
            const bool ok = b.step > a.step && deep == (kind == LBM_PASS_DEEP) && roll == (kind == LBM_PASS_ROLLING) &&
                            strip == (kind == LBM_PASS_STRIPS);
            static const char *names[4] = {"tiles", "deep", "rolling", "strips"};
            std::printf("%s%d%s ", names[kind], cycles, ok ? "" : "?");
            n -= cycles;
        }
        std::printf("\n");
        lbm_destroy(c);
        std::free(ws);
    }
    return 0;
}
