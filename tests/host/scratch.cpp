// What the library's host code asks of the runtime, without a device: memory
// that calls share between them, and launches.  One scenario a run, by name;
// 0 if it holds.
#include "fake_hip.h"

#include <cmath>
#include <vector>

#include "shadow_accrual.h"

namespace {

int bad = 0;

#define CHECK(c)                                                            \
    do {                                                                    \
        if (!(c)) {                                                         \
            std::printf("line %d: %s does not hold\n", __LINE__, #c);       \
            ++bad;                                                          \
        }                                                                   \
    } while (0)
// a call of the library that succeeds
#define OK(ctx, c)                                                                        \
    do {                                                                                  \
        if ((c) != SA_OK) {                                                               \
            std::printf("line %d: %s: %s\n", __LINE__, #c, sa_last_error(ctx));           \
            ++bad;                                                                        \
        }                                                                                 \
    } while (0)

template <class T>
T *device(size_t n)
{
    void *p = nullptr;
    (void)hipMalloc(&p, sizeof(T) * (n ? n : 1));
    return (T *)p;
}

// n unit squares a hundred metres apart, whose order on the device is their own.
sa_scene *upload(sa_ctx *ctx, int n)
{
    std::vector<int32_t> off;
    std::vector<float> xy, h(n, 10.f);
    for (int b = 0; b <= n; ++b) off.push_back(4 * b);
    for (int b = 0; b < n; ++b)
        for (const auto &c : {std::pair<float, float>{0, 0}, {1, 0}, {1, 1}, {0, 1}}) {
            xy.push_back(100.f * (b % 200) + c.first);
            xy.push_back(100.f * (b / 200) + c.second);
        }
    sa_scene *s = nullptr;
    fake::rt().read = [n](void *d, size_t bytes) {
        int32_t *w = (int32_t *)d;
        if (bytes == sizeof(int32_t) * (size_t)n)  // the ranks
            for (int b = 0; b < n; ++b) w[b] = b;
        else if (bytes == 64 * (size_t)(n - 1))  // the nodes: a chain, words 10 and 11 the children
            for (int b = 0; b < n - 1; ++b) {
                w[16 * b + 10] = ~b;
                w[16 * b + 11] = b < n - 2 ? b + 1 : ~(n - 1);
            }
        else
            return false;
        return true;
    };
    OK(ctx, sa_scene_upload(ctx, n, off.data(), xy.data(), h.data(), &s));
    fake::rt().read = nullptr;
    return s;
}

// `days` days at the given steps, a bin each, or all in one.
sa_path *upload_path(sa_ctx *ctx, int days, double step, double seg, bool one_bin = false)
{
    const sa_site site{40.7, -74.0, -5.0};
    const sa_timespan span{2019, 1, 1, days, 480.0, 960.0, step, seg, 0};
    sa_sunpath_buf b{};
    CHECK(sa_sunpath(&site, &span, &b) == SA_OK);
    std::vector<int32_t> so(days + 1), ko(days + 1), bin(days);
    std::vector<double> t(b.n_samples), d(3 * b.n_samples), w(b.n_samples), kt(b.n_knots), kd(3 * b.n_knots);
    b.cap_days = days;
    b.cap_samples = b.n_samples;
    b.cap_knots = b.n_knots;
    b.day_sample_off = so.data();
    b.t_min = t.data();
    b.dir = d.data();
    b.weight = w.data();
    b.day_knot_off = ko.data();
    b.knot_t = kt.data();
    b.knot_dir = kd.data();
    CHECK(sa_sunpath(&site, &span, &b) == SA_OK);
    b.day_bin = one_bin ? bin.data() : nullptr;
    sa_path *p = nullptr;
    OK(ctx, sa_path_upload(ctx, &b, &p));
    return p;
}

// Long height edits stage their arrays in memory of their own, whatever a
// region score does with its weights in between.
void edit_score()
{
    sa_ctx *ctx = nullptr;
    CHECK(sa_create(0, nullptr, &ctx) == SA_OK);
    const size_t before = fake::rt().live.size();
    sa_scene *s = upload(ctx, 100);
    sa_path *one = upload_path(ctx, 1, 5.0, 30.0), *five = upload_path(ctx, 5, 5.0, 30.0);
    std::vector<int32_t> ids(80);
    std::vector<float> h(80, 20.f);
    for (int k = 0; k < 80; ++k) ids[k] = k;
    float *v = device<float>(5 * 10);
    int64_t *off = device<int64_t>(2);
    double *out = device<double>(1);
    const double w[5] = {1, 1, 1, 1, 1};
    OK(ctx, sa_scene_set_heights(ctx, s, 80, ids.data(), h.data()));
    OK(ctx, sa_region_score(ctx, one, v, 10, w, off, 1, nullptr, out));
    OK(ctx, sa_scene_set_heights(ctx, s, 80, ids.data(), h.data()));
    OK(ctx, sa_region_score(ctx, five, v, 10, w, off, 1, nullptr, out));
    OK(ctx, sa_scene_set_heights(ctx, s, 80, ids.data(), h.data()));
    sa_path_destroy(one);
    sa_path_destroy(five);
    sa_scene_destroy(s);
    CHECK(fake::rt().live.size() > before);
    sa_destroy(ctx);
    CHECK(fake::rt().live.size() == 3);  // the test's own
}

// A call on n points of a context's scene and path.
struct Calls {
    sa_ctx *ctx = nullptr;
    sa_scene *scene = nullptr;
    sa_path *path = nullptr;
    static constexpr int kMost = 5000000, kVariants = 4;
    float *x = device<float>(kMost), *minutes = device<float>(kMost), *var_h = device<float>(kVariants);
    int32_t *counts = device<int32_t>(kMost), *var_ids = device<int32_t>(kVariants);
    int64_t *var_off = device<int64_t>(kVariants + 1);

    Calls(int prisms, int days, double seg, double step = 30.0, bool one_bin = true)
    {
        OK(ctx, sa_create(0, nullptr, &ctx));
        scene = upload(ctx, prisms);
        path = upload_path(ctx, days, step, seg, one_bin);
    }
    ~Calls()
    {
        sa_path_destroy(path);
        sa_scene_destroy(scene);
        sa_destroy(ctx);
    }
    sa_points points(int64_t n) const { return sa_points{n, x, x, x, nullptr, nullptr, nullptr}; }
    void accrual(int64_t n)
    {
        const sa_points p = points(n);
        const sa_accum_opts o{SA_ACCRUAL, 0, 1.f, 0, nullptr, nullptr, nullptr};
        OK(ctx, sa_accumulate(ctx, scene, &p, path, &o, counts, minutes, nullptr));
    }
    void sampled(int64_t n, float *longest = nullptr)
    {
        const sa_points p = points(n);
        const sa_accum_opts o{SA_SAMPLED, 0, 1.f, 0, nullptr, longest, nullptr};
        OK(ctx, sa_accumulate(ctx, scene, &p, path, &o, counts, minutes, nullptr));
    }
    void raster(int64_t n, int64_t max_texels = 0)
    {
        const sa_points p = points(n);
        const sa_sam_opts o{2.f, 0.1f, {0, 0, 0, 2000, 2000, 20}, 0, 1.f, max_texels};
        OK(ctx, sa_sam_accumulate(ctx, scene, &p, path, &o, counts, minutes));
    }
    void gradient(int64_t n)
    {
        const sa_points p = points(n);
        OK(ctx, sa_grad_heights(ctx, scene, &p, path, nullptr, nullptr, minutes));
    }
    void sums(int64_t n)
    {
        OK(ctx, sa_region_sum(ctx, minutes, n, var_off, 3, nullptr, (double *)x));
    }
    void batched(int64_t n)
    {
        const sa_points p = points(n);
        const sa_accum_opts o{SA_ACCRUAL, 0, 1.f, 0, nullptr, nullptr, nullptr};
        OK(ctx, sa_accumulate_batched(ctx, scene, kVariants, 1, var_ids, var_h, &p, var_off, path, &o, counts, minutes));
    }
};

// After an eager call of a size, calls of that size or less can be captured:
// nothing waits, is allocated or freed; and eager ones leave the memory a graph
// was captured over.
void capture()
{
    for (const bool batched : {false, true})
        for (const int64_t first : {(int64_t)100000, (int64_t)Calls::kMost}) {  // in pieces, and too large for them
            Calls c(100, 2, 30.0);
            auto call = [&](int64_t n) { batched ? c.batched(n) : c.accrual(n); };
            call(first);
            const int frees = fake::rt().frees;
            fake::rt().capturing = true;
            for (const int64_t n : {100000, 90000, 64, 1}) call(n);
            fake::rt().capturing = false;
            for (const int64_t n : {90000, 1, 100000}) call(n);
            CHECK(fake::rt().frees == frees);
        }
    // without an eager call first, calls that need memory are refused, and the
    // capture is as it was
    Calls c(100, 2, 30.0);
    const sa_points p = c.points(1000);
    const sa_accum_opts o{SA_ACCRUAL, 0, 1.f, 0, nullptr, nullptr, nullptr};
    fake::rt().capturing = true;
    CHECK(sa_accumulate(c.ctx, c.scene, &p, c.path, &o, c.counts, c.minutes, nullptr) == SA_ERR_OOM);
    CHECK(sa_accumulate_batched(c.ctx, c.scene, c.kVariants, 1, c.var_ids, c.var_h, &p, c.var_off, c.path, &o, c.counts,
                                c.minutes) == SA_ERR_OOM);
    CHECK(sa_grad_heights(c.ctx, c.scene, &p, c.path, nullptr, nullptr, c.minutes) == SA_ERR_OOM);
    CHECK(sa_region_sum(c.ctx, c.minutes, 1000, c.var_off, 3, nullptr, (double *)c.x) == SA_ERR_OOM);
    fake::rt().capturing = false;
    c.accrual(1000);
    c.batched(1000);
    c.gradient(1000);
    c.sums(1000);
    fake::rt().capturing = true;
    c.accrual(1000);
    c.batched(1000);
    c.gradient(1000);
    c.sums(1000);
    fake::rt().capturing = false;
}

// Where the memory a call would like cannot be had, the first call finds that
// out and every later one takes what is there: no wait, no allocation tried, no
// buffer given up.
void short_of_memory()
{
    fake::Runtime &r = fake::rt();
    const size_t kMiB = 1 << 20;
    auto settled = [&](auto call) {
        call();
        const int refused = r.refused, mallocs = r.mallocs, frees = r.frees, syncs = r.syncs;
        CHECK(refused > 0);
        call();
        call();
        CHECK(r.refused == refused && r.mallocs == mallocs && r.frees == frees && r.syncs == syncs);
        r.refused = 0;
        r.limit = SIZE_MAX;
    };
    for (const size_t limit : {600 * kMiB, 300 * kMiB}) {  // the views: half the wish, or the least
        Calls c(20000, 20, 5.0);
        r.limit = limit;
        settled([&]() { c.accrual(1000000); });
    }
    {  // and the sums of pieces beside them
        Calls c(100, 2, 30.0);
        r.limit = 100 * kMiB;
        settled([&]() { c.accrual(1000); });
    }
    for (const bool masks : {false, true}) {  // the sampled form's views, or its masks
        Calls c(masks ? 100 : 20000, masks ? 3 : 20, 5.0);
        r.limit = 4 * kMiB;
        const int packets = fake::launches("k_sampled_q"), fans = fake::launches("k_sampled_fan");
        settled([&]() { c.sampled(1000000); });
        CHECK(fake::launches("k_sampled_q") == packets + 3 && fake::launches("k_sampled_fan") == fans);
        c.sampled(1);  // a size not refused
        CHECK(fake::launches("k_sampled_fan") > fans);
    }
    {  // the second raster map
        Calls a(100, 1, 30.0), b(100, 1, 30.0);
        r.largest = 0;
        a.raster(1000);
        r.limit = r.largest - 1;
        const int clears = fake::launches("k_sam_clear");
        settled([&]() { b.raster(1000); });
        CHECK(fake::launches("k_sam_clear") == clears + 1);
    }
    {  // which a caller's cap counts too
        Calls a(100, 1, 30.0), b(100, 1, 30.0);
        r.largest = 0;
        a.raster(1000);
        const size_t two = r.largest;
        r.largest = 0;
        b.raster(1000, (int64_t)(two / 4) - 8192);  // (less the points' bounds: one and not quite two)
        CHECK(r.largest < two * 6 / 10 && r.largest > two * 4 / 10);
    }
}

// The sampled form's views and masks stay within 256 MiB each, however many
// instants a path has and however few prisms a scene.
void fan_masks()
{
    for (const double step : {1.0, 0.1}) {
        Calls c(20, step < 1.0 ? 40 : 365, 60.0, step);
        for (const int64_t n : {(int64_t)1, (int64_t)20000, (int64_t)Calls::kMost})
            for (const bool longest : {false, true}) {
                fake::rt().largest = 0;
                c.sampled(n, longest ? c.minutes : nullptr);
                CHECK(fake::rt().largest <= 256u << 20);
            }
    }
    CHECK(fake::launches("k_sampled_fan") > 0 && fake::launches("k_sampled_q") == 0);
}

// More bins in a launch than a grid has rows: 192 years, a bin a day, in pieces.
void many_bins()
{
    Calls c(2, 70000, 30.0, 480.0, false);
    const int sums = fake::launches("k_add_pieces");
    c.accrual(1);
    CHECK(fake::launches("k_add_pieces") >= sums + 3);
}

// Only the sun's height is checked at upload: whatever its horizontal part, the
// directions that order the views' entries are finite and at most one, or two
// entries could be given one place and another's be left as it was.
void sun_without_direction()
{
    sa_ctx *ctx = nullptr;
    OK(ctx, sa_create(0, nullptr, &ctx));
    for (const double x : {(double)NAN, (double)INFINITY, -1e300, 1e39, 3.0}) {
        int32_t so[2] = {0, 1}, ko[2] = {0, 2};
        double t[1] = {0}, w[1] = {1}, kt[2] = {0, 2};
        double d[3] = {x, x, 0.5}, kd[6] = {x, 0.2, 0.5, 0.3, 0.3, 0.6};
        sa_sunpath_buf b{};
        b.n_days = 1;
        b.n_samples = 1;
        b.n_knots = std::isnan(x) ? 0 : 2;  // coincident directions are refused, and a NaN makes them so
        ko[1] = b.n_knots;
        b.day_sample_off = so;
        b.day_knot_off = ko;
        b.t_min = t;
        b.dir = d;
        b.weight = w;
        b.knot_t = kt;
        b.knot_dir = kd;
        const auto before = fake::rt().live;
        sa_path *p = nullptr;
        OK(ctx, sa_path_upload(ctx, &b, &p));
        int seen = 0;
        for (const auto &a : fake::rt().live) {
            // a chunk of instants: a line, the direction at words 8 and 9; a segment: two, at 30 and 31
            if (before.count(a.first) || (a.second != 64 && a.second != 128)) continue;
            const float *f = (const float *)a.first + (a.second == 64 ? 8 : 30);
            CHECK(std::fabs(f[0]) <= 1.f && std::fabs(f[1]) <= 1.f);
            ++seen;
        }
        CHECK(seen >= (b.n_knots ? 3 : 1));  // (two copies of the segment)
        sa_path_destroy(p);
    }
    sa_destroy(ctx);
}

}  // namespace

int main(int argc, char **argv)
{
    const std::map<std::string, void (*)()> all = {{"edit_score", edit_score}, {"capture", capture}, {"short_of_memory", short_of_memory},
                                                       {"sun_without_direction", sun_without_direction},
                                                       {"fan_masks", fan_masks}, {"many_bins", many_bins}};
    const auto it = all.find(argc > 1 ? argv[1] : "");
    if (it == all.end()) {
        std::printf("no such scenario\n");
        return 2;
    }
    it->second();
    bad += fake::rt().faults;
    std::printf("%s: %s\n", it->first.c_str(), bad ? "FAILED" : "holds");
    return bad ? 1 : 0;
}
