// Which march the library's host code gives a frame or a batch: the queue
// launches of the host-memory HIP stand-in are recorded, and scenes on either
// side of every line of the rule checked.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "dpvr.h"
#include "dpvr_kernels.h"
#include "tet_kernels.h"

// the stand-in's queue and mesh launchers under other names, so that these can
// look at the launches they check
#define launch_march_queue launch_march_queue_checked
#define launch_tet_frame launch_tet_frame_checked
namespace dpvr {
hipError_t launch_march_queue_checked(const QueueParams& q, StorageK storage, int workgroups, hipStream_t stream);
hipError_t launch_tet_frame_checked(TetFrameParams f, int stages, hipStream_t stream);
}
#include "fake_hip.cpp"
#undef launch_march_queue
#undef launch_tet_frame

static std::vector<int> g_staged[2];       // per storage: the launches' staged flags
static int g_alone = -1, g_tet_tiles = 0;
namespace dpvr {
hipError_t launch_tet_frame(TetFrameParams f, int stages, hipStream_t stream) {
    if (stages & kTetMarch) {
        g_alone = f.alone;
        g_tet_tiles = f.total_tiles;
    }
    return launch_tet_frame_checked(f, stages, stream);
}
hipError_t launch_march_queue(const QueueParams& q, StorageK storage, int workgroups, hipStream_t stream) {
    g_staged[storage == kF16 ? 1 : 0].push_back(q.staged);
    return launch_march_queue_checked(q, storage, workgroups, stream);
}
}  // namespace dpvr

static int g_fail = 0;
#define EXPECT(cond)                                                             \
    do {                                                                         \
        if (!(cond)) {                                                           \
            std::printf("FAILED line %d: %s\n", __LINE__, #cond);               \
            ++g_fail;                                                            \
        }                                                                        \
    } while (0)

static void* buf(size_t bytes) {
    void* p = nullptr;
    if (posix_memalign(&p, 256, bytes ? bytes : 256) != 0) std::abort();
    return p;
}

// A grid of count[0] x count[1] x count[2] bricks of ext voxels each, seen from twice its
// longest edge (az, el in degrees, 45 degrees high) by an image 4/3 as wide as
// high.  The stand-in touches neither voxels nor images, so every brick and
// partial shares one small buffer.
struct Scene {
    int32_t ext[3], count[3];
    double step;
    int f16, height;
    double az = 30.0, el = 20.0;
};

struct Setup {
    vr_context ctx = nullptr;
    std::vector<vr_brick> bricks;
    std::vector<vr_partial> parts;
    void* ws;
    void* img;
    vr_camera_desc cam{};

    explicit Setup(const Scene& s) {
        EXPECT(vr_context_create(0, nullptr, &ctx) == VR_OK);
        img = buf(4096);
        EXPECT(vr_set_transfer_function(ctx, static_cast<float*>(img), DPVR_TF_ENTRIES, 0.f, 1.f, 1.f) == VR_OK);
        EXPECT(vr_set_render_params(ctx, s.step, 0.f) == VR_OK);
        double dims[3], top = 0.0;
        for (int c = 0; c < 3; ++c) top = std::fmax(top, dims[c] = (double)s.ext[c] * s.count[c]);
        const double pi = std::acos(-1.0), a = s.az * pi / 180.0, e = s.el * pi / 180.0;
        const double off[3] = {std::cos(e) * std::sin(a), std::sin(e), std::cos(e) * std::cos(a)};
        double eye[3], tgt[3];
        const double up[3] = {0, 1, 0};
        for (int c = 0; c < 3; ++c) {
            tgt[c] = 0.5 * dims[c];
            eye[c] = tgt[c] + 2.0 * top * off[c];
        }
        EXPECT(vr_set_camera_perspective(ctx, eye, tgt, up, 45.0, s.height * 4 / 3, s.height) == VR_OK);
        cam.kind = 0;
        for (int c = 0; c < 3; ++c) {
            cam.eye[c] = eye[c];
            cam.target[c] = tgt[c];
            cam.up[c] = up[c];
        }
        cam.fovy_deg = 45.0;
        cam.width = s.height * 4 / 3;
        cam.height = s.height;
        const double sp[3] = {1, 1, 1};
        size_t bytes = 0;
        EXPECT(vr_brick_workspace_size(s.ext, 1, s.f16 ? VR_F16 : VR_F32, &bytes) == VR_OK);
        for (int k = 0; k < s.count[2]; ++k)
            for (int j = 0; j < s.count[1]; ++j)
                for (int i = 0; i < s.count[0]; ++i) {
                    const double lo[3] = {(double)i * s.ext[0], (double)j * s.ext[1], (double)k * s.ext[2]};
                    vr_brick b = nullptr;
                    EXPECT(vr_brick_create(ctx, s.ext, 1, lo, sp, s.f16 ? VR_F16 : VR_F32, img, bytes, &b) == VR_OK);
                    EXPECT(vr_brick_set_data(b, static_cast<float*>(img)) == VR_OK);
                    bricks.push_back(b);
                    int32_t r[4];
                    EXPECT(vr_partial_roi(ctx, b, r) == VR_OK);
                    parts.push_back(vr_partial{r[0], r[1], r[2], r[3], static_cast<float*>(img),
                                               static_cast<float*>(img), nullptr});
                }
        EXPECT(vr_frame_workspace_size((int32_t)bricks.size(), &bytes) == VR_OK);
        ws = buf(bytes);
    }
    ~Setup() {
        for (vr_brick b : bricks) EXPECT(vr_brick_release(b) == VR_OK);
        EXPECT(vr_context_release(ctx) == VR_OK);
        std::free(ws);
        std::free(img);
    }
    // 1 staged, 0 direct
    int frame(int f16) {
        g_staged[0].clear();
        g_staged[1].clear();
        size_t bytes = 0;
        EXPECT(vr_frame_workspace_size((int32_t)bricks.size(), &bytes) == VR_OK);
        EXPECT(vr_render_partials(ctx, (int32_t)bricks.size(), bricks.data(), parts.data(), ws, bytes) == VR_OK);
        EXPECT(g_staged[f16].size() == 1 && g_staged[1 - f16].empty());
        return g_staged[f16].empty() ? -1 : g_staged[f16][0];
    }
    int batch(int f16) {
        g_staged[0].clear();
        g_staged[1].clear();
        const vr_tf_desc tf{static_cast<float*>(img), 0.f, 1.f, 1.f, 0};
        std::vector<vr_batch_job> jobs;
        for (size_t i = 0; i < bricks.size(); ++i) jobs.push_back(vr_batch_job{bricks[i], 0, 0, parts[i]});
        size_t bytes = 0;
        EXPECT(vr_batch_workspace_size((int32_t)jobs.size(), 0, &bytes) == VR_OK);
        void* bws = buf(bytes);
        vr_batch b = nullptr;
        EXPECT(vr_batch_create(ctx, 1, &cam, 1, &tf, (int32_t)jobs.size(), jobs.data(), 0, nullptr, bws, bytes, &b) ==
               VR_OK);
        const int r = g_staged[f16].empty() ? -1 : g_staged[f16].back();
        if (b) EXPECT(vr_batch_release(b) == VR_OK);
        std::free(bws);
        return r;
    }
};

// A unit cube of cells^3 cells cut into tetrahedra per part, `copies` of it
// over each other (each its own part), filling an image of the given size; 1 if
// a wavefront takes a tile.
static int tet_route(int copies, int width, int height, double dt, int* tiles, int cells = 1) {
    const int n = cells + 1, step[3] = {n * n, n, 1};
    const int order[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
    std::vector<double> v;
    std::vector<int32_t> t;
    for (int i = 0; i < n * n * n; ++i)
        for (int c = 0; c < 3; ++c) v.push_back((double)(i / step[c] % n) / cells);
    for (int i = 0; i < n * n * n; ++i) {
        if (i / step[0] == cells || i / step[1] % n == cells || i % n == cells) continue;
        for (const auto& o : order) {
            int32_t w = i;
            t.push_back(w);
            for (int c : o) t.push_back(w += step[c]);
        }
    }
    vr_context ctx = nullptr;
    EXPECT(vr_context_create(0, nullptr, &ctx) == VR_OK);
    void* img = buf((size_t)16 * width * height);
    EXPECT(vr_set_transfer_function(ctx, static_cast<float*>(img), DPVR_TF_ENTRIES, 0.f, 1.f, 1.f) == VR_OK);
    EXPECT(vr_set_render_params(ctx, dt, 0.f) == VR_OK);
    const double pos[3] = {0.5, 0.5, -1}, dir[3] = {0, 0, 1}, up[3] = {0, 1, 0};
    EXPECT(vr_set_camera_orthographic(ctx, pos, dir, up, 0.5, width, height) == VR_OK);
    std::vector<vr_tetpart> parts;
    std::vector<void*> mem;
    const std::vector<float> vals(v.size() / 3);
    for (int i = 0; i < copies; ++i) {
        vr_tetpart q = nullptr;
        EXPECT(vr_tetpart_create(ctx, v.data(), (int32_t)(v.size() / 3), t.data(), (int32_t)(t.size() / 4), &q) == VR_OK);
        double lo[3], hi[3];
        int32_t grid[3];
        int64_t count;
        size_t bytes = 0;
        int32_t nt = 0;
        EXPECT(vr_tetpart_info(q, lo, hi, grid, &count, &bytes, &nt) == VR_OK);
        mem.push_back(buf(bytes));
        EXPECT(vr_tetpart_attach(q, mem.back(), bytes) == VR_OK);
        EXPECT(vr_tetpart_set_values(q, vals.data()) == VR_OK);
        parts.push_back(q);
    }
    size_t need = 0;
    EXPECT(vr_tetparts_workspace_size(ctx, copies, parts.data(), 1, &need) == VR_OK);
    mem.push_back(buf(need));
    const float bg[4] = {0, 0, 0, 0};
    EXPECT(vr_render_tetparts(ctx, copies, parts.data(), 1, bg, mem.back(), need, static_cast<float*>(img), nullptr) ==
           VR_OK);
    for (vr_tetpart q : parts) EXPECT(vr_tetpart_release(q) == VR_OK);
    EXPECT(vr_context_release(ctx) == VR_OK);
    for (void* p : mem) std::free(p);
    std::free(img);
    *tiles = g_tet_tiles;
    return g_alone;
}

int main() {
    // a frame of few tiles marches from HBM by default; a caller's choice of
    // the staged march, as a path or as a configuration, is taken as it is
    const Scene small{{64, 64, 64}, {1, 1, 1}, 0.5, 0, 160};
    for (int f16 = 0; f16 < 2; ++f16) {
        Scene s = small;
        s.f16 = f16;
        { Setup u(s); EXPECT(u.frame(f16) == 0 && u.batch(f16) == 0); }
        {
            Setup u(s);
            EXPECT(vr_set_march_path(u.ctx, VR_PATH_STAGED) == VR_OK);
            EXPECT(u.frame(f16) == 1 && u.batch(f16) == 1);
            EXPECT(vr_set_march_path(u.ctx, VR_PATH_DIRECT) == VR_OK);
            EXPECT(u.frame(f16) == 0);
            EXPECT(vr_set_march_path(u.ctx, VR_PATH_STAGED) == VR_OK);
            EXPECT(u.frame(f16) == 1);
        }
        {
            Setup u(s);
            EXPECT(vr_set_march_config(u.ctx, f16 ? VR_F16 : VR_F32, VR_STAGING_RING, 16, 8) == VR_OK);
            EXPECT(u.frame(f16) == 1 && u.batch(f16) == 1);
            EXPECT(vr_set_march_path(u.ctx, VR_PATH_DIRECT) == VR_OK);
            EXPECT(u.frame(f16) == 0);
        }
    }
    // on either side of the rule's lines (voxels a pixel in brackets)
    const struct {
        Scene s;
        int staged;
    } lines[] = {
        {{{200, 200, 200}, {1, 1, 1}, 0.5, 0, 400}, 0},              // 506 tiles of one brick
        {{{200, 200, 200}, {3, 3, 3}, 0.5, 0, 96}, 0},               // 158 tiles, 32 MB bricks [10.4]
        {{{200, 200, 200}, {3, 3, 3}, 0.5, 0, 160}, 1},              // 347 tiles [6.2]
        {{{100, 100, 100}, {5, 5, 5}, 0.5, 0, 110}, 1},              // 500 tiles, 4 MB bricks [7.5]
        {{{48, 48, 48}, {7, 7, 7}, 0.5, 0, 74}, 0},                  // 362 tiles, 0.5 MB bricks [7.5]
        {{{32, 32, 32}, {8, 8, 8}, 0.25, 0, 106}, 0},                // 919 tiles, 0.16 MB bricks [4.0]
        {{{64, 64, 64}, {6, 6, 6}, 0.5, 0, 289}, 0},                 // 1.2 MB bricks [2.2]
        {{{64, 64, 64}, {6, 6, 6}, 0.25, 0, 212}, 1},                // [3.0]
        {{{64, 64, 64}, {6, 6, 6}, 0.5, 0, 116}, 1},                 // [5.5]
        {{{80, 80, 80}, {6, 6, 6}, 0.5, 0, 497}, 0},                 // 2.2 MB bricks [1.6]
        {{{80, 80, 80}, {6, 6, 6}, 0.5, 0, 199}, 1},                 // [4.0]
        {{{100, 100, 100}, {5, 5, 5}, 0.5, 0, 690}, 0},              // 4.2 MB bricks [1.2]
        {{{100, 100, 100}, {5, 5, 5}, 0.5, 0, 376}, 1},              // [2.2]
        {{{192, 192, 128}, {2, 2, 2}, 0.5, 0, 1080}, 0},             // 19 MB bricks [0.59]
        {{{256, 256, 256}, {2, 2, 2}, 0.5, 0, 1082}, 0},             // 69 MB bricks [0.78]
        {{{256, 256, 256}, {2, 2, 2}, 0.5, 0, 1082, 30.0, 60.0}, 1},
        {{{256, 256, 256}, {2, 2, 2}, 0.5, 0, 2120}, 0},             // [0.4]
        {{{250, 900, 500}, {1, 1, 1}, 1.0, 0, 1345}, 1},             // 456 MB [1.11]
        {{{250, 900, 500}, {1, 1, 1}, 0.5, 0, 2485}, 0},             // [0.6]
        {{{250, 900, 500}, {1, 1, 1}, 0.5, 0, 2485, 30.0, 60.0}, 1},
        {{{2300, 1100, 40}, {1, 1, 1}, 1.0, 0, 3432}, 1},            // slices of 10 MB [1.11]
        {{{256, 512, 256}, {4, 2, 2}, 0.5, 0, 1080}, 1},             // 16 bricks of 1024 x 1024 x 512 at full HD
        {{{128, 128, 128}, {2, 2, 2}, 0.5, 0, 2000, 100.0, 20.0}, 0},
        {{{64, 64, 64}, {6, 6, 6}, 0.5, 1, 397}, 0},                 // float16, 0.6 MB bricks [1.6]
        {{{64, 64, 64}, {6, 6, 6}, 0.5, 1, 800}, 1},                 // [0.8]
        {{{125, 125, 125}, {4, 4, 4}, 0.5, 1, 376}, 0},              // 4.1 MB bricks [2.2]
        {{{125, 125, 125}, {4, 4, 4}, 0.25, 1, 517}, 1},             // [1.6]
        {{{80, 80, 80}, {6, 6, 6}, 0.25, 1, 199}, 0},                // 1.1 MB bricks [4.0]
        {{{80, 80, 80}, {6, 6, 6}, 0.25, 1, 106}, 1},                // [7.5]
        {{{158, 158, 158}, {4, 4, 4}, 0.5, 1, 475}, 1},              // 8.2 MB bricks [2.2]
        {{{80, 80, 80}, {6, 6, 6}, 0.5, 1, 662}, 0},                 // 1.1 MB bricks [1.2]
        {{{80, 80, 80}, {6, 6, 6}, 0.5, 1, 662, 30.0, 60.0}, 1},
        {{{125, 125, 125}, {4, 4, 4}, 0.25, 1, 330}, 0},             // 4.1 MB bricks [2.5]
        {{{64, 64, 64}, {6, 6, 6}, 0.5, 1, 530}, 0},                 // 0.6 MB bricks [1.2]
        {{{64, 64, 64}, {6, 6, 6}, 0.25, 1, 475}, 1},                // [1.3]
        {{{64, 64, 64}, {6, 6, 6}, 0.25, 1, 289}, 0},                // [2.2]
        {{{64, 64, 64}, {6, 6, 6}, 1.0, 1, 530}, 0},                 // [1.2]
        // along y, pixel rows along z (and along x)
        {{{100, 100, 100}, {5, 5, 5}, 0.5, 0, 690, 90.0, 60.0}, 1},  // 4.2 MB bricks [1.2]
        {{{100, 100, 100}, {5, 5, 5}, 0.5, 0, 690, 0.0, 60.0}, 0},
        {{{64, 64, 64}, {6, 6, 6}, 0.5, 0, 289, 90.0, 60.0}, 1},     // 1.2 MB bricks [2.2]
        {{{256, 256, 256}, {2, 2, 2}, 0.5, 0, 2120, 90.0, 60.0}, 1}, // 69 MB bricks [0.4]
    };
    for (const auto& c : lines) {
        Setup u(c.s);
        const int frame = u.frame(c.s.f16), batch = u.batch(c.s.f16);
        if (frame != c.staged || batch != c.staged) {
            std::printf("FAILED: %d x %d x %d in %d bricks of an axis, step %g, storage %d, height %d: frame %d, batch "
                        "%d, expected %d\n", c.s.ext[0], c.s.ext[1], c.s.ext[2], c.s.count[0], c.s.step, c.s.f16,
                        c.s.height, frame, batch, c.staged);
            ++g_fail;
        }
    }
    // tetrahedral tiles by wavefront: many, or fewer with few samples across a part
    {
        int tiles = 0;
        EXPECT(tet_route(1, 640, 640, 0.25, &tiles) == 0 && tiles == 6400);
        EXPECT(tet_route(1, 800, 800, 0.2, &tiles) == 1 && tiles == 10000);
        EXPECT(tet_route(1, 800, 800, 0.125, &tiles) == 0 && tiles == 10000);
        EXPECT(tet_route(2, 904, 904, 0.01, &tiles) == 0 && tiles == 25538);
        EXPECT(tet_route(3, 800, 800, 0.01, &tiles) == 1 && tiles == 30000);
        // 827,052 tetrahedra in all: from 37,546 tiles on
        EXPECT(tet_route(2, 1080, 1080, 0.01, &tiles, 41) == 0 && tiles == 36450);
        EXPECT(tet_route(2, 1120, 1120, 0.01, &tiles, 41) == 1 && tiles == 39200);
    }
    std::printf("%s: %d failed expectations\n", g_fail ? "FAIL" : "OK", g_fail);
    return g_fail ? 1 : 0;
}
