// Host allocations of the library that fail: a call in which the k-th fails
// returns SC_ENOMEM, for k = 0, 1, ... (every one of the first 16, then in
// steps of a sixteenth) until it succeeds, and no exception leaves it.  host_memory_check <mechanism> load|plan.  The operator
// new below replaces the library's (its calls from the library's own code are
// counted, other libraries' are not).
#include <hip/hip_runtime_api.h>

#include <dlfcn.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "stiffchem.h"

static long left = -1;  // allocations until one fails; negative: none does

void *operator new(size_t n)
{
    Dl_info who;
    if (left >= 0 && dladdr(__builtin_return_address(0), &who) && std::strstr(who.dli_fname, "libstiffchem") && left-- == 0)
        throw std::bad_alloc();
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

// call() until it succeeds, its k-th allocation failing; returns the last k, or
// -1 where a failure was not reported as one
template <class F, class G>
static long every_failure(const char *what, F call, G empty)
{
    for (long k = 0;; k += 1 + k / 16) {
        left = k;
        const sc_status s = call();
        left = -1;
        if (s == SC_OK) return k;
        if (s != SC_ENOMEM || !empty()) {
            std::printf("%s: allocation %ld: status %d, %s\n", what, k, s, sc_last_error());
            return -1;
        }
    }
}

int main(int argc, char **argv)
{
    if (argc != 3) return 2;
    std::string text;
    std::FILE *f = std::fopen(argv[1], "rb");
    if (!f) return 2;
    for (int c; (c = std::fgetc(f)) != EOF;) text.push_back((char)c);
    std::fclose(f);
    sc_mech *m = nullptr;
    const bool load = !std::strcmp(argv[2], "load");
    const long loads = load ? every_failure(
                                  "sc_mech_load", [&] { return sc_mech_load(text.data(), text.size(), &m); },
                                  [&] { return m == nullptr; })
                            : sc_mech_load(text.data(), text.size(), &m) == SC_OK ? 0 : -1;
    if (loads < 0) return 1;
    std::printf("load %ld\n", loads);
    if (load) {
        sc_mech_free(m);
        return 0;
    }
    size_t before = 0, after = 0, total = 0;
    sc_plan *p = nullptr;
    sc_options o;
    sc_default_options(&o);
    o.linalg = SC_LINALG_SPARSE;
    o.thermo_tol = 1e-3;  // a small table, quickly fitted
    o.thermo_degree = 3;
    o.thermo_Tmin = 1000.0;
    o.thermo_Tmax = 1100.0;
    if (sc_plan_create(m, 0, &o, &p) != SC_OK) return 1;  // the device's own first allocations
    sc_plan_free(p);
    p = nullptr;
    if (hipMemGetInfo(&before, &total) != hipSuccess) return 1;
    const long plans = every_failure("sc_plan_create", [&] { return sc_plan_create(m, 0, &o, &p); }, [&] { return p == nullptr; });
    if (plans < 0) return 1;
    sc_mech_info info;
    sc_mech_info_get(m, &info);
    std::vector<double> fuel(info.n_species, 0.0), ox(info.n_species, 0.0);
    fuel[0] = 1.0;
    ox[1] = 1.0;
    const sc_mapping map = {0.1, 10.0, 0.0};
    const long maps = every_failure("sc_plan_set_mapping", [&] { return sc_plan_set_mapping(p, fuel.data(), ox.data(), &map); },
                                    [] { return true; });
    if (maps < 0) return 1;
    sc_plan_free(p);
    if (hipMemGetInfo(&after, &total) != hipSuccess) return 1;
    std::printf("plan %ld mapping %ld device bytes kept %lld\n", plans, maps, (long long)before - (long long)after);
    sc_mech_free(m);
    return 0;
}
