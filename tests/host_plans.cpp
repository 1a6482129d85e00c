// The library's host-side planning, reached from the tests: the planning
// functions are internal to nlos_abi.cpp, which is compiled in here; the kernel
// launchers it names come from the library and are never called.
#include "nlos_abi.cpp"

// Plan of the pair kernel for a call alone (solo) or a list's request with a
// share of `target` workgroups: unit, pair, threads of a workgroup of one unit,
// workgroups per split, split, windows, workgroups, LDS bytes.
extern "C" int host_forward_plan(const nlos_params* p, int32_t n_patches, int64_t target, int32_t solo, int64_t* out)
{
    float taps[nlos::kMaxTaps];
    int32_t R = 0;
    int rc = jitter_taps(p->fwhm_ps, p->bin_ps, taps, &R);
    if (rc != NLOS_OK) return rc;
    nlos::Plan plan;
    rc = make_plan(p, n_patches, R, target, solo ? PlanFor::alone : PlanFor::list, &plan);
    if (rc != NLOS_OK) return rc;
    const int64_t v[10] = {plan.tl, plan.tx, plan.ty, plan.pair, plan.one, plan.groups, plan.n_split, plan.n_tw,
                           plan.n_blocks, (int64_t)plan.lds_bytes};
    std::memcpy(out, v, sizeof(v));
    return NLOS_OK;
}

// Plan of the smooth forward: moment rows per scan point (0: by taps), tile,
// tiles, splits, workgroups, workgroups per CU (moments), bytes of the kernels' table.
extern "C" int host_smooth_plan(const nlos_params* p, int32_t n_patches, int64_t* out)
{
    nlos::SmoothArgs a;
    int rc = smooth_setup(p, nullptr, 0, nullptr, &a);
    if (rc != NLOS_OK) return rc;
    SmoothPlan sp;
    int split = 1;
    rc = smooth_plan(p, n_patches, a.Rs, &sp, &split);
    if (rc != NLOS_OK) return rc;
    const int64_t v[8] = {sp.moments, sp.tx, sp.ty, sp.tiles, split, sp.n_blocks, sp.wg, (int64_t)sp.taps_bytes};
    std::memcpy(out, v, sizeof(v));
    return NLOS_OK;
}

// Plan of the adjoint: correlation rows per scan point (0: by taps), scan points
// per stage, splits, patch blocks, two row buffers, bytes ahead of the partials,
// LDS bytes.
extern "C" int host_adjoint_plan(const nlos_params* p, int32_t n_patches, int64_t* out)
{
    nlos::SmoothArgs a;
    int rc = smooth_setup(p, nullptr, 0, nullptr, &a);
    if (rc != NLOS_OK) return rc;
    AdjPlan ap;
    rc = adjoint_plan(p, n_patches, a.Rs, &ap);
    if (rc != NLOS_OK) return rc;
    const int64_t v[7] = {ap.moments, ap.rows, ap.split, ap.pbk, ap.dbuf, (int64_t)ap.c_bytes, (int64_t)ap.lds};
    std::memcpy(out, v, sizeof(v));
    return NLOS_OK;
}

// Launches of the noise sampler over n elements: their number; the largest one's threads.
extern "C" int64_t host_noise_launches(int64_t n, int64_t* threads)
{
    const int tile = nlos::noise_tile(n);
    int64_t count = 0;
    *threads = 0;
    for (int64_t first = 0; first < n; ++count) {
        const int64_t m = nlos::noise_launch(n - first, tile);
        *threads = std::max<int64_t>(*threads, (m + tile - 1) / tile * nlos::kNoiseBlock);
        first += m;
    }
    return count;
}

// The smooth kernels' polynomials at width sigma (bins), with one term more for
// the adjoint: their terms (0: by taps), nodes and coefficients.
extern "C" int host_moment_fit(double sigma, int32_t adjoint, double* node, double* coef)
{
    int n = nlos::smooth_moments(sigma);
    if (n == 0) return 0;
    if (adjoint) n = nlos::adj_moments(n);
    const nlos::MomentFit f = moment_fit(sigma, (int)std::ceil(6.0 * sigma), n);
    for (int m = 0; m < n; ++m) {
        node[m] = f.node[m];
        for (int j = 0; j < n; ++j) coef[m * n + j] = f.coef[m * nlos::kMaxMoments + j];
    }
    return n;
}
