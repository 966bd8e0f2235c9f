// Which plans run two chains of launches, seen from the host: the launches of
// a step on the library's own streams, with abi_stubs.cpp in place of the HIP
// runtime and the kernels (no device pointer is dereferenced).  Built with
// -fsanitize=undefined, so that the lines between the forms are the library's.
#include <stdint.h>
#include <string.h>

#include "../../include/diffus.h"
#include "abi_stubs.cpp"

namespace {
int failures = 0;

void expect(bool ok, const char *what, int i = 0)
{
    if (!ok) {
        fprintf(stderr, "FAILED: %s %d (%s)\n", what, i, dus_last_error());
        ++failures;
    }
}

template <typename T>
T *dev(uintptr_t a)
{
    return reinterpret_cast<T *>(a);
}

const uintptr_t kZ = 0x1000000, kPoses = 0x2000000, kImg = 0x3000000, kGrad = 0x4000000, kWs = 0x5000000;

struct Plan {
    dus_plan *p = nullptr;
    int64_t ws = 0;
    uintptr_t img = kImg;
    int flags;

    // fans of rays x samples, n of them; blur on
    Plan(std::vector<std::vector<int>> kinds, int fl, int blur = 1) : flags(fl)
    {
        dus_volume v;
        memset(&v, 0, sizeof(v));
        v.nx = v.ny = v.nz = 64;
        for (int a = 0; a < 3; ++a) v.spacing_mm[a] = 1.0f;
        dus_physics ph;
        memset(&ph, 0, sizeof(ph));
        ph.spk_cell = 8;
        ph.blur_on = blur;
        ph.blur_sigma0 = 0.5f;
        ph.blur_sigma1 = 2.0f;
        std::vector<dus_fan> f;
        int64_t off = 0;
        for (const auto &k : kinds)
            for (int i = 0; i < k[0]; ++i) {
                f.push_back(dus_fan{k[1], k[2], 1.0f, 0.25f, 0.0f, (int32_t)f.size(), off});
                off += (int64_t)k[1] * k[2];
            }
        expect(dus_plan_create(&p, &v, f.data(), (int32_t)f.size(), &ph, flags) == DUS_OK, "create");
        ws = dus_plan_workspace_bytes(p);
    }

    ~Plan() { dus_plan_destroy(p); }

    // (a new image pointer: a plan with a graph captures it again)
    int step()
    {
        img += 0x1000;
        return dus_plan_step(p, dev<float>(kZ), dev<float>(kPoses), dev<float>(kImg + 0x800000), dev<float>(img),
                             dev<double>(kGrad), (flags & DUS_PLAN_POSE_ONLY) ? nullptr : dev<float>(kGrad + 0x200000),
                             dev<float>(kGrad + 0x100000), dev<void>(kWs), (size_t)ws, nullptr);
    }

    long launches()
    {
        const long l0 = stub_launches();
        expect(step() == DUS_OK, "step");
        return stub_launches() - l0;
    }

    // whether a step launches on two streams, and whether from a graph
    bool two()
    {
        const long a = on_others();
        expect(step() == DUS_OK, "step");
        return on_others() > a;
    }

    bool graph()
    {
        for (Obj *t : g_streams) t->was_origin = false;
        expect(step() == DUS_OK, "step");
        bool captured = false;
        for (Obj *t : g_streams) captured = captured || t->was_origin;
        return captured;
    }

    static long on_others()
    {
        long n = 0;
        for (Obj *t : g_streams)
            if (!t->was_origin) n += t->ops;
        return n;
    }

    // every launch of a step failing in turn: reported, nothing left unjoined
    void fail_each()
    {
        const long n = launches();
        for (long k = 1; k <= n; ++k) {
            stub_fail_launch(k);
            expect(step() == DUS_EHIP, "failed launch reported", (int)k);
            stub_fail_launch(0);
            expect(stub_unjoined_captures() == 0, "capture ended with every fork joined", (int)k);
            expect(stub_open_work() == 0, "no work left unjoined", (int)k);
            expect(step() == DUS_OK, "step after a failed one", (int)k);
        }
    }
};

// launches of a full step with image and blur: five a table, and the end
const long kOne = 6, kTwo = 11, kPoseOne = 5, kPoseTwo = 9;
}  // namespace

int main()
{
    for (int flags : {0, (int)DUS_PLAN_NO_GRAPH}) {
        // the smallest plans, and the line of 3 * 2^20 ray-samples
        expect(Plan({{2, 1, 2}}, flags).launches() == kOne, "smallest");
        expect(Plan({{4, 5, 100}}, flags).launches() == kOne, "small");
        expect(Plan({{3, 524, 2000}}, flags).launches() == kOne, "below the line");
        expect(Plan({{3, 525, 2000}}, flags).launches() == kTwo, "above the line");
        expect(Plan({{1, 2000, 2000}}, flags).launches() == kOne, "one fan");
        expect(Plan({{3, 525, 2000}}, flags | DUS_PLAN_ONE_STREAM).launches() == kOne, "one stream");
        expect(Plan({{3, 524, 2000}}, flags | DUS_PLAN_POSE_ONLY).launches() == kPoseOne, "pose only, below");
        expect(Plan({{3, 525, 2000}}, flags | DUS_PLAN_POSE_ONLY).launches() == kPoseTwo, "pose only, above");
        // many small fans: past one table with dL/dZ, past six with poses alone
        expect(!Plan({{64, 8, 64}}, flags).two(), "one table");
        expect(Plan({{65, 8, 64}}, flags).two(), "two tables");
        expect(!Plan({{65, 8, 64}}, flags | DUS_PLAN_DETERMINISTIC).two(), "two tables, deterministic");
        expect(!Plan({{65, 8, 64}}, flags | DUS_PLAN_ONE_STREAM).two(), "two tables, one stream");
        expect(!Plan({{65, 8, 64}, {200, 0, 64}}, flags | DUS_PLAN_POSE_ONLY).two(), "empty fans");
        expect(!Plan({{384, 8, 64}}, flags | DUS_PLAN_POSE_ONLY).two(), "six tables, pose only");
        expect(Plan({{385, 8, 64}}, flags | DUS_PLAN_POSE_ONLY).two(), "seven tables, pose only");
        expect(!Plan({{65, 8, 64}}, flags).graph(), "no graph for small fans");
        expect(Plan({{3, 525, 2000}}, flags).graph() == (flags == 0), "graph above the line");
        // long rays: beside others on the second stream (from a graph), unless
        // they are few or many, or no others are there
        const std::vector<std::vector<int>> beside = {{2, 100, 5000}, {8, 256, 1000}};
        expect(Plan(beside, flags).launches() == kOne && Plan(beside, flags).graph() == (flags == 0), "long beside short");
        expect(!Plan(beside, flags | DUS_PLAN_ONE_STREAM).graph(), "long beside short, one stream");
        expect(Plan({{1, 20, 5000}, {3, 200, 300}}, flags).graph() == (flags == 0), "few long beside many short");
        expect(Plan(beside, flags | DUS_PLAN_DETERMINISTIC).graph() == (flags == 0), "long beside short, deterministic");
        expect(!Plan({{3, 525, 2000}}, flags | DUS_PLAN_DETERMINISTIC).graph(), "deterministic");
        for (std::vector<int> k : {std::vector<int>{1, 64, 5000}, {12, 256, 5000}, {2, 256, 8000}, {1, 512, 9000}}) {
            Plan p({k}, flags);
            expect(p.launches() == kOne && !p.two() && !p.graph(), "long rays alone", k[0] * k[1]);
            // without spans they are rays like others
            dus_schedule sc = {0, 0, 0, 0, -1};
            expect(dus_plan_set_schedule(p.p, &sc) == DUS_OK, "schedule");
            expect(p.launches() == (k[0] > 1 ? kTwo : kOne), "long rays, no spans", k[0] * k[1]);
            // tiles and chunks that few rays cannot share, and an explicit length
            sc = {16, 8, 0, 0, 4000};
            expect(dus_plan_set_schedule(p.p, &sc) == DUS_OK, "schedule");
            expect(p.launches() == kOne && !p.graph(), "long rays alone, explicit", k[0] * k[1]);
        }
        // equal fans split into two groups of no more tables than they need
        for (int n : {65, 127, 128, 129, 192, 255, 256, 257})
            expect(Plan({{n, 8, 64}}, flags).launches() == 5 * (n <= 128 ? 2 : n == 129 ? 3 : n <= 256 ? 4 : 5) + 1,
                   "tables of", n);
        Plan({{4, 5, 100}}, flags).fail_each();
        Plan({{130, 5, 100}}, flags).fail_each();
        Plan({{3, 525, 2000}}, flags).fail_each();
    }
    if (failures) {
        fprintf(stderr, "%d failures\n", failures);
        return 1;
    }
    printf("chains driver: ok\n");
    return 0;
}
