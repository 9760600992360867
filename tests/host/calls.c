/* Whole calls of the library on the stand-in HIP runtime (hip_stub.h): what
 * they allocate, wait for and hand on.  One scenario per argument. */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "hip_stub.h"
#include "pet_os.h"

int hipGetLastError(void);

static int A_, B_, C_;
#define A ((void*)&A_)
#define B ((void*)&B_)
#define C ((void*)&C_)
static float buf[16];       /* stands for the caller's device buffers (no kernel runs) */

#define CHECK(c)                                                       \
    do {                                                               \
        if (!(c)) {                                                    \
            printf("line %d: %s (%s)\n", __LINE__, #c, pet_os_last_error()); \
            exit(1);                                                   \
        }                                                              \
    } while (0)

static pet_os_geom* geometry(int n, int nz, int angles, int rd, int subsets) {
    pet_os_geom_desc d;
    memset(&d, 0, sizeof(d));
    d.dim = nz > 1 ? 3 : 2;
    d.nx = d.ny = n;
    d.nz = nz;
    d.vx = d.vy = d.ds = 2.0;
    d.vz = d.ring_pitch = nz > 1 ? 2.5 : 1.0;
    d.n_angles = angles;
    d.n_radial = 3 * n / 2 + 1;
    d.n_rings = nz;
    d.max_ring_diff = rd;
    d.det_radius = 2.0 * n;
    d.n_subsets = subsets;
    pet_os_geom* g = NULL;
    CHECK(pet_os_create_geometry(&d, &g) == PET_OS_OK);
    return g;
}

static pet_os_params params(void) {
    pet_os_params p;
    memset(&p, 0, sizeof(p));
    p.mode = PET_OS_BSREM;
    p.beta = 0.1;
    p.gamma_R = 2.0;
    p.eps = 1e-12;
    p.U = 1e3;
    p.t_clip = 1e-4;
    p.lambda0 = 1.0;
    p.a = 0.25;
    p.objective_every = 1;
    return p;
}

/* A gradient that finds no memory for its sinogram gives back what it took;
 * the next call may not use it while another stream's work does. */
static void failed_call(void) {
    pet_os_geom* g = geometry(64, 16, 64, 3, 8);
    pet_os_params p = params();
    double phi;
    CHECK(pet_os_back(g, buf, 0, buf, A) == PET_OS_OK);
    void* used = stub_last_malloc;
    CHECK(stub_pending(A));
    stub_limit = stub_live;
    CHECK(pet_os_subset_gradient(g, &p, buf, buf, buf, 0, buf, B) == PET_OS_ERR_OUT_OF_MEMORY);
    stub_limit = (size_t)1 << 34;
    hipGetLastError();
    const long waits = stub_stream_waits;
    stub_last_copy = NULL;
    CHECK(pet_os_objective(g, &p, buf, buf, buf, &phi, C) == PET_OS_OK);
    CHECK(stub_last_copy != NULL);
    CHECK(stub_block(stub_last_copy) != used || !stub_pending(A) || stub_stream_waits > waits);
}

/* What whole calls keep is bounded over all geometries, yields to the library's
 * own allocations and goes with the last geometry. */
static void memory_kept(void) {
    enum { N = 24 };
    pet_os_geom* g[N];
    pet_os_params p = params();
    double phi;
    const size_t before = stub_live;
    size_t tables = 0;
    for (int k = 0; k < N; ++k) {
        g[k] = geometry(128 + 2 * k, 16, 60, 3, 8);
        tables += stub_block_bytes(stub_last_malloc);
    }
    for (int k = 0; k < N; ++k) {
        CHECK(pet_os_forward(g[k], buf, 0, buf, A) == PET_OS_OK);
        CHECK(pet_os_objective(g[k], &p, buf, buf, buf, &phi, A) == PET_OS_OK);
        CHECK(pet_os_subset_gradient(g[k], &p, buf, buf, buf, 0, buf, B) == PET_OS_OK);
        CHECK(pet_os_back(g[k], buf, 1, buf, C) == PET_OS_OK);
    }
    CHECK(stub_live - tables - before <= (size_t)256 << 20);
    CHECK(stub_live - tables - before > (size_t)1 << 20);
    /* no memory left but what is kept: a geometry's tables get it */
    stub_limit = stub_live;
    pet_os_geom* one = geometry(128, 16, 60, 3, 8);
    stub_limit = (size_t)1 << 34;
    CHECK(pet_os_destroy_geometry(one) == PET_OS_OK);
    for (int k = 0; k < N; ++k) CHECK(pet_os_destroy_geometry(g[k]) == PET_OS_OK);
    CHECK(stub_live == before);
}

/* Calls on one stream don't wait for what another has queued, on the device or
 * on the host, although they use scratch of the same sizes. */
static void streams(void) {
    pet_os_geom* g = geometry(64, 16, 64, 3, 8);
    pet_os_params p = params();
    double phi;
    for (int n = 0; n < 3; ++n) {
        CHECK(pet_os_back(g, buf, 0, buf, A) == PET_OS_OK);
        CHECK(pet_os_back(g, buf, 0, buf, B) == PET_OS_OK);
    }
    CHECK(stub_stream_waits == 0 && stub_host_waits == 0 && stub_pending(A) && stub_pending(B));
    CHECK(pet_os_objective(g, &p, buf, buf, buf, &phi, C) == PET_OS_OK);
    CHECK(pet_os_forward(g, buf, 0, buf, C) == PET_OS_OK);
    CHECK(pet_os_subset_gradient(g, &p, buf, buf, buf, 0, buf, C) == PET_OS_OK);
    CHECK(pet_os_reconstruct(g, &p, buf, buf, buf, 1, NULL, C) == PET_OS_OK);
    CHECK(stub_stream_waits == 0 && stub_pending(A) && stub_pending(B));
    /* and a stream's own calls go on without more and more memory */
    const long mallocs = stub_mallocs;
    for (int n = 0; n < 20; ++n) CHECK(pet_os_back(g, buf, 0, buf, A) == PET_OS_OK);
    CHECK(stub_mallocs - mallocs <= 3 && stub_stream_waits == 0);
}

/* A back-projection is asynchronous whatever memory there is: where the kept
 * blocks are all in use it takes the kernel that needs none. */
static void asynchronous(void) {
    enum { N = 40 };
    static int s[N];
    pet_os_geom* g = geometry(256, 16, 60, 3, 1);
    const size_t before = stub_live;
    for (int k = 0; k < N; ++k) {
        CHECK(pet_os_back(g, buf, 0, buf, &s[k]) == PET_OS_OK);
        CHECK(stub_pending(&s[k]));
    }
    CHECK(stub_host_waits == 0 && stub_stream_waits == 0 && stub_frees == 0);
    CHECK(stub_live - before <= (size_t)256 << 20);
    const int columns = stub_launches_of("k_bp3I"), quads = stub_launches_of("k_bp3q");
    CHECK(columns > 0 && quads > 0);
    /* no memory at all */
    for (int k = 0; k < N; ++k) stub_finish(&s[k]);
    pet_os_geom* h = geometry(400, 16, 60, 3, 1);
    stub_limit = stub_live;
    CHECK(pet_os_back(h, buf, 0, buf, A) == PET_OS_OK);
    CHECK(stub_pending(A) && stub_host_waits == 0 && stub_frees == 0);
}

/* A back-projection does not break the capture of another stream. */
static void beside_a_capture(void) {
    pet_os_geom* g = geometry(64, 16, 64, 3, 8);
    stub_capturing = 1;
    for (int n = 0; n < 5; ++n) CHECK(pet_os_back(g, buf, 0, buf, A) == PET_OS_OK);
    CHECK(stub_capture_breaks == 0);
}

/* A batch whose step fails keeps its count: the steps queued before it are
 * counted, and its updates are not queued again. */
static void failed_step(void) {
    enum { N = 2, STEPS = 12 };
    static float y[1 << 20];
    pet_os_geom* g[N] = {geometry(64, 1, 60, 0, 4), geometry(64, 16, 24, 3, 4)};
    pet_os_params p = params();
    const char* forward[] = {"k_fp_batch", "k_fp3q_batch"};
    const char* update[] = {"k_bp_batch", "k_upd3_batch"};
    for (int bad = 0; bad < 13; ++bad) {
        pet_os_batch* b = NULL;
        int32_t slot, active;
        int64_t left, was[2];
        CHECK(pet_os_batch_create(4, &b) == PET_OS_OK);
        for (int k = 0; k < N; ++k) CHECK(pet_os_batch_add(b, g[k], &p, y, y, y, 3, A, &slot) == PET_OS_OK);
        CHECK(pet_os_batch_step(b, 1, A) == PET_OS_OK);
        for (int k = 0; k < N; ++k) was[k] = stub_launches_of(update[k]) - 1;
        const int f0 = stub_launches_of(forward[0]) - 1;
        /* launch number `bad` of the next ones fails */
        stub_fail_launch = stub_launches + bad;
        CHECK(pet_os_batch_step(b, 2, A) == PET_OS_ERR_DEVICE);
        stub_fail_launch = -1;
        hipGetLastError();
        CHECK(pet_os_batch_slot_status(b, 0, &active, &left) == PET_OS_OK);
        const int done = stub_launches_of(update[0]) - (int)was[0], dun = stub_launches_of(update[1]) - (int)was[1];
        const int steps = done < dun ? done : dun;
        CHECK(left == STEPS - steps);
        /* to the end: every update once */
        CHECK(pet_os_batch_run(b, A) == PET_OS_OK);
        CHECK(pet_os_batch_slot_status(b, 1, &active, &left) == PET_OS_OK && left == 0 && !active);
        for (int k = 0; k < N; ++k) CHECK(stub_launches_of(update[k]) - was[k] == STEPS);
        CHECK(stub_launches_of(forward[0]) - f0 >= STEPS);
        CHECK(pet_os_batch_destroy(b) == PET_OS_OK);
    }
}

/* Images of more rows than a grid's y and z hold, and rays of more angles and
 * bins than a launch of a block each. */
static void large_grids(void) {
    pet_os_geom_desc d;
    memset(&d, 0, sizeof(d));
    d.dim = 3;
    d.nx = 3;
    d.ny = 70001;
    d.nz = d.n_rings = 33;
    d.vx = d.vy = d.ds = 2.0;
    d.vz = d.ring_pitch = 2.5;
    d.n_angles = 8;
    d.n_radial = 301;
    d.max_ring_diff = 1;
    d.det_radius = 1e5;
    d.n_subsets = 2;
    pet_os_geom* g = NULL;
    pet_os_params p = params();
    double phi;
    CHECK(pet_os_create_geometry(&d, &g) == PET_OS_OK);
    CHECK(pet_os_back(g, buf, 0, buf, A) == PET_OS_OK && stub_launches_of("k_turn3") == 1);
    CHECK(pet_os_subset_gradient(g, &p, buf, buf, buf, 1, buf, A) == PET_OS_OK && stub_launches_of("k_turn3") == 2);
    CHECK(pet_os_objective(g, &p, buf, buf, buf, &phi, A) == PET_OS_OK);
    CHECK(pet_os_reconstruct(g, &p, buf, buf, buf, 1, NULL, A) == PET_OS_OK);
    d.nx = d.ny = 40;
    d.nz = d.n_rings = 4;
    d.n_angles = 8200;
    d.n_radial = 1101;
    d.max_ring_diff = 0;
    d.n_subsets = 4;
    int64_t nnz;
    CHECK(pet_os_create_geometry(&d, &g) == PET_OS_OK);
    CHECK(pet_os_forward(g, buf, 0, buf, A) == PET_OS_OK);
    CHECK(pet_os_objective(g, &p, buf, buf, buf, &phi, A) == PET_OS_OK);
    CHECK(pet_os_nnz(g, 0, &nnz) == PET_OS_OK);
}

/* The 3D autotuner times only shapes that subiterations can use. */
static void autotune(void) {
    int32_t now[4], def[4];
    pet_os_geom* g = geometry(64, 16, 64, 3, 8);        /* by quads */
    const long before = stub_launches, mallocs = stub_mallocs;
    CHECK(pet_os_autotune(g, 1, A) == PET_OS_OK);
    CHECK(stub_launches == before && stub_mallocs == mallocs);
    CHECK(pet_os_geometry_shapes(g, now, def) == PET_OS_OK && !memcmp(now, def, sizeof(now)));
    pet_os_geom* deep = geometry(24, 70, 24, 3, 8);     /* not */
    const long made = stub_launches;
    CHECK(pet_os_autotune(deep, 1, A) == PET_OS_OK && stub_launches > made);
}

/* Memory for the subset sinogram bin by bin, but not as quads, is enough. */
static void memory_limits(void) {
    pet_os_geom* g = geometry(32, 24, 64, 23, 1);
    pet_os_params p = params();
    const size_t compact = (size_t)64 * 24 * 24 * 49 * 4, quads = (size_t)4 * 64 * 24 * 25 * 24 * 4;
    const size_t images = (size_t)5 * 32 * 32 * 24 * 4 + (1 << 20);
    CHECK(quads > compact + images);
    const size_t limit = stub_live + compact + images;
    const int columns = stub_launches_of("k_bp3I");
    stub_limit = limit;
    pet_os_state* st = NULL;
    CHECK(pet_os_state_create(g, &p, &st) == PET_OS_OK);
    hipGetLastError();
    CHECK(pet_os_subiteration(st, buf, buf, buf, A) == PET_OS_OK && stub_launches_of("k_bp3I") == columns + 1);
    CHECK(pet_os_state_destroy(st) == PET_OS_OK);
    CHECK(pet_os_reconstruct(g, &p, buf, buf, buf, 1, NULL, A) == PET_OS_OK);
    CHECK(stub_launches_of("k_bp3I") == columns + 2);
    CHECK(pet_os_subset_gradient(g, &p, buf, buf, buf, 1, buf, A) == PET_OS_OK);
    CHECK(stub_launches_of("k_bp3I") == columns + 3);
    const pet_os_geom* gs[1] = {g};
    float* fs[1] = {buf};
    const float* ys[1] = {buf};
    const int32_t n[1] = {1};
    CHECK(pet_os_reconstruct_batch(1, gs, &p, fs, ys, ys, n, A) == PET_OS_OK);
    CHECK(stub_launches_of("k_bp3_batch") == 1 && stub_launches_of("k_bp3q") == 0);
    stub_limit = (size_t)1 << 34;
    CHECK(pet_os_reconstruct(g, &p, buf, buf, buf, 1, NULL, A) == PET_OS_OK && stub_launches_of("k_bp3q") == 1);
}

int main(int argc, char** argv) {
    static const struct { const char* name; void (*run)(void); } all[] = {
        {"failed_call", failed_call}, {"memory_kept", memory_kept}, {"streams", streams},
        {"asynchronous", asynchronous}, {"beside_a_capture", beside_a_capture},
        {"failed_step", failed_step}, {"large_grids", large_grids},
        {"autotune", autotune}, {"memory_limits", memory_limits}};
    for (size_t k = 0; argc > 1 && k < sizeof(all) / sizeof(all[0]); ++k)
        if (!strcmp(argv[1], all[k].name)) {
            all[k].run();
            printf("ok\n");
            return 0;
        }
    printf("no such scenario\n");
    return 2;
}
