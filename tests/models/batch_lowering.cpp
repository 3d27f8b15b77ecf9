// dl_batch_copy on the host, with its executors replaced by ones that write down what they are given: what a batch of copies is
// lowered to, whichever of the lowerings it takes, against what the batch means, and what that costs.
#include "../../paper_2511_06605_amd/csrc/dl_api.hip"

#include <stdio.h>

#include <chrono>
#include <map>
#include <random>
#include <set>
#include <tuple>

namespace {
std::vector<dl_plan_item> g_done;  // what the executors were given, as items
bool g_keep = true;
}  // namespace

int dl_exec_plain(const dl_plain_item *items, size_t n, hipStream_t, const dl_arm *, bool *launched)
{
    for (size_t i = 0; i < n && g_keep; ++i) g_done.push_back({items[i].src, items[i].bytes, 1, 0, {items[i].dst}});
    *launched = true;
    return DL_OK;
}
int dl_exec_fused(const dl_fused_item *items, size_t n, hipStream_t, const dl_arm *, bool *launched)
{
    const dl_plan_item *it = reinterpret_cast<const dl_plan_item *>(items);
    if (g_keep) g_done.insert(g_done.end(), it, it + n);
    *launched = true;
    return DL_OK;
}
// Beyond the lowering nothing is asked for.
int dl_exec_swap(const dl_swap_item *, size_t, hipStream_t, const dl_arm *, bool *) { return DL_ERR_STATE; }
int dl_exec_init() { return DL_ERR_STATE; }
int dl_exec_shutdown() { return DL_OK; }
int dl_static_init(int) { return DL_ERR_STATE; }
bool dl_device_error_pending() { return false; }
int dl_dispatch_on_device(const void *const *, void *const *, int, const uint32_t *, size_t, const uint8_t *, uint64_t, hipStream_t, bool *) { return DL_ERR_STATE; }
bool dl_armed_ready() { return true; }
int dl_armed_begin(dl_arm *arm, hipStream_t *)
{
    arm->nowait = g_dl.mode == DL_MODE_PRELAUNCH ? 0u : 1u;
    return DL_OK;
}
void dl_armed_commit(uint32_t, bool, bool) {}
int dl_standby_try(const dl_plan_item *, size_t, bool *taken)
{
    *taken = false;
    return DL_OK;
}
int dl_standby_enter() { return DL_OK; }
int dl_standby_leave() { return DL_OK; }
extern "C" int dl_prelaunch_stop(void) { return DL_OK; }
extern "C" uint64_t dl_last_ticket(void) { return 0; }
extern "C" int dl_wait(uint64_t, uint64_t) { return DL_OK; }

namespace {

#define CHECK(cond, ...)                                \
    do {                                                \
        if (!(cond)) {                                  \
            printf("line %d: %s: ", __LINE__, #cond);   \
            printf(__VA_ARGS__);                        \
            printf("\n");                               \
            return false;                               \
        }                                               \
    } while (0)

using copy_key = std::tuple<uint64_t, uint64_t, uint64_t>;
void *at(uint64_t a) { return (void *)a; }

// What the items move, one entry per destination.
std::multiset<copy_key> moves(const std::vector<dl_plan_item> &items)
{
    std::multiset<copy_key> m;
    for (const dl_plan_item &it : items)
        for (uint32_t j = 0; j < it.k; ++j) m.insert({(uint64_t)it.src, (uint64_t)it.dst[j], it.bytes});
    return m;
}

// The items of `desc` as the header states them: empty and identical copies left out, copies of one range together in order of
// first appearance, at most DL_PLAN_FANOUT destinations each; or one by one.
std::vector<dl_plan_item> expected(const std::vector<dl_copy_desc> &desc, bool infer)
{
    std::vector<dl_plan_item> items;
    std::map<std::pair<const void *, size_t>, size_t> open;
    for (const dl_copy_desc &d : desc) {
        if (d.bytes == 0 || d.src == d.dst) continue;
        const auto key = std::make_pair((const void *)d.src, d.bytes);
        const auto f = open.find(key);
        if (infer && f != open.end() && items[f->second].k < (uint32_t)DL_PLAN_FANOUT) {
            dl_plan_item &it = items[f->second];
            it.dst[it.k++] = d.dst;
            continue;
        }
        open[key] = items.size();
        items.push_back({d.src, d.bytes, 1, 0, {d.dst}});
    }
    return items;
}

bool same(const std::vector<dl_plan_item> &a, const std::vector<dl_plan_item> &b)
{
    return a.size() == b.size() && std::equal(a.begin(), a.end(), b.begin(), [](const dl_plan_item &x, const dl_plan_item &y) {
               return x.src == y.src && x.bytes == y.bytes && x.k == y.k && std::equal(x.dst, x.dst + DL_PLAN_FANOUT, y.dst);
           });
}

// The batch through dl_batch_copy in every mode that lowers it, with and without inference, validated or not.
bool check(const std::vector<dl_copy_desc> &desc, const char *what)
{
    bool null = false;
    for (const dl_copy_desc &d : desc) null = null || (d.bytes && (!d.src || !d.dst));
    for (const int mode : {DL_MODE_ONESHOT, DL_MODE_PRELAUNCH, DL_MODE_SIGNAL, DL_MODE_STANDBY, DL_MODE_AUTO})
        for (const bool infer : {false, true})
            for (const int validate : {0, 1}) {
                g_dl.mode = mode;
                g_dl.cfg.infer_broadcast = infer;
                g_dl.validate = validate;
                g_done.clear();
                const int rc = dl_batch_copy(desc.data(), desc.size(), nullptr);
                CHECK(rc == (null ? DL_ERR_INVALID : DL_OK), "%s, %zu copies, mode %d, infer %d: status %d", what, desc.size(), mode, infer, rc);
                if (null) {
                    CHECK(g_done.empty(), "%s: refused, but %zu items were executed", what, g_done.size());
                    continue;
                }
                const std::vector<dl_plan_item> want = expected(desc, infer && desc.size() > 1);
                CHECK(moves(g_done) == moves(want), "%s, %zu copies, mode %d, infer %d", what, desc.size(), mode, infer);
                CHECK(same(g_done, want), "%s, %zu copies, mode %d, infer %d: other items", what, desc.size(), mode, infer);
            }
    return true;
}

bool lists()
{
    std::mt19937_64 rng(7);
    uint64_t to = 1ull << 40;  // a fresh destination for every copy, so that no list overlaps itself
    const auto dst = [&] { return at(to += 1u << 20); };
    if (!check({}, "empty")) return false;
    if (!check({{at(4096), dst(), 16}}, "one")) return false;
    for (const size_t n : {2u, 3u, 15u, 16u, 17u, 63u, 64u, 65u, 300u, 1100u}) {
        std::vector<dl_copy_desc> distinct, prefixes, shared;
        for (size_t i = 0; i < n; ++i) {
            distinct.push_back({at((i + 1) << 24), dst(), 4096});
            prefixes.push_back({at(1u << 24), dst(), 1 + i});
            shared.push_back({at((1 + rng() % (n / 2 + 1)) << 24), dst(), 1000 + rng() % 2});
        }
        if (!check(distinct, "distinct") || !check(prefixes, "prefixes of one source") || !check(shared, "shared sources")) return false;
        // one repeated range, first met at any place; then a tenth and a twentieth destination for it
        for (const size_t where : {(size_t)1, n / 2, n - 1}) {
            std::vector<dl_copy_desc> l = distinct;
            l[where].src = l[0].src;
            if (!check(l, "a repeated range")) return false;
            for (int more = 0; more < 20; ++more) l.push_back({l[0].src, dst(), 4096});
            if (!check(l, "a range repeated 20 times more")) return false;
        }
        // empty and identical copies, also with null pointers, which are looked at in copies that move something only
        for (const bool repeated : {false, true}) {
            std::vector<dl_copy_desc> l = repeated ? shared : distinct;
            for (int q = 0; q < 6; ++q) l.insert(l.begin() + rng() % (l.size() + 1), dl_copy_desc{q & 1 ? nullptr : at(64), q & 2 ? nullptr : at(128), 0});
            for (int q = 0; q < 3; ++q) l.insert(l.begin() + rng() % (l.size() + 1), dl_copy_desc{at(512 + q), at(512 + q), 100});
            if (!check(l, "empty and identical")) return false;
            for (const size_t where : {(size_t)0, l.size() / 2, l.size() - 1})
                for (const bool src : {false, true}) {
                    std::vector<dl_copy_desc> bad = l;
                    bad[where] = {src ? nullptr : at(1u << 30), src ? dst() : nullptr, 8};
                    if (!check(bad, "a null pointer")) return false;
                }
        }
    }
    return true;
}

double best_us(const std::vector<dl_copy_desc> &desc, int times)
{
    double best = 1e30;
    for (int t = 0; t < times; ++t) {
        const auto t0 = std::chrono::steady_clock::now();
        dl_batch_copy(desc.data(), desc.size(), nullptr);
        best = std::min(best, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count());
    }
    return best;
}

double best_inferred_us(const std::vector<dl_copy_desc> &desc, int times)
{
    std::vector<dl_plan_item> items(desc.size());
    double best = 1e30;
    for (int t = 0; t < times; ++t) {
        const auto t0 = std::chrono::steady_clock::now();
        dl_plan_batch_inferred(desc.data(), desc.size(), items.data(), items.size());
        best = std::min(best, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count());
    }
    return best;
}

// Linear in the number of copies, whatever they have in common; and a range that is met again late costs no second beginning
// (three times the inference alone at 16 000 copies; a fifth more without).
bool cost(bool print)
{
    g_dl.mode = DL_MODE_ONESHOT;
    g_dl.validate = 0;
    g_dl.cfg.infer_broadcast = 1;
    g_keep = false;
    for (const size_t n : {256u, 512u, 1000u, 16000u, 100000u}) {
        std::vector<dl_copy_desc> distinct, prefixes;
        for (size_t i = 0; i < n; ++i) {
            distinct.push_back({at(((i * 2654435761u) % 1000003u + 1) << 16), at((i + 1) << 40), 65536});
            prefixes.push_back({at(1u << 24), at((i + 1) << 40), 1 + i});
        }
        std::vector<dl_copy_desc> last = distinct;
        last[n - 1].src = last[0].src;
        const int times = n <= 1000 ? 2000 : 20;
        const double d = best_us(distinct, times), l = best_us(last, times), p = best_us(prefixes, n <= 1000 ? 200 : 1);
        if (print) printf("%zu copies: distinct %.2f us, the last one's source repeated %.2f, prefixes of one source %.2f\n", n, d, l, p);
        double ratio = 1e30;
        for (int attempt = 0; attempt < 5 && ratio > 2.0; ++attempt) ratio = std::min(ratio, best_us(last, times) / best_inferred_us(last, times));
        if (print) printf("  the last one's source repeated, against the inference alone: %.2f\n", ratio);
        if (!print && n == 16000) CHECK(ratio < 2.0, "%zu copies, the last one's source repeated: %.2f times the inference alone", n, ratio);
        if (!print) CHECK(p < 20.0 * d + 1000.0, "%zu prefixes of one source %.0f us, distinct copies %.0f", n, p, d);
    }
    return true;
}

}  // namespace

int main(int argc, char **)
{
    g_dl.inited = true;
    if (argc > 1) return cost(true) ? 0 : 1;
    if (!lists() || !cost(false)) return 1;
    printf("ok\n");
    return 0;
}
