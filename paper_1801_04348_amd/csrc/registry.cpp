// Registry of compiled kernel instances and their resource usage.  The
// instance lists and the resource figures (taken from the compiler's
// kernel-resource-usage report at build time) are generated by build.py.
#include <cstring>
#include <functional>
#include <string>
#include <unordered_map>

#include "pk_internal.hpp"

extern "C" const pkk::KernelEntry *pk_gen_entries(int *n);
struct pk_gen_resource {
    const char *name;
    int vgpr, agpr, sgpr, scratch, lds, occupancy;
};
extern "C" const pk_gen_resource *pk_gen_resources(int *n);

namespace pk {

const std::vector<KernelEntry> &registry() {
    static const std::vector<KernelEntry> reg = [] {
        int n = 0;
        const KernelEntry *e = pk_gen_entries(&n);
        return std::vector<KernelEntry>(e, e + n);
    }();
    return reg;
}

const KernelResources *resources_of(const char *name) {
    static const std::unordered_map<std::string, KernelResources> res = [] {
        std::unordered_map<std::string, KernelResources> m;
        int n = 0;
        const pk_gen_resource *r = pk_gen_resources(&n);
        for (int i = 0; i < n; ++i)
            m[r[i].name] = KernelResources{r[i].vgpr, r[i].agpr, r[i].sgpr, r[i].scratch, r[i].lds, r[i].occupancy};
        return m;
    }();
    auto it = res.find(name);
    return it == res.end() ? nullptr : &it->second;
}

const KernelResources *resources_of(const KernelEntry &e) {
    static const std::vector<const KernelResources *> by_index = [] {
        std::vector<const KernelResources *> v;
        for (const auto &x : registry()) v.push_back(resources_of(x.name));
        return v;
    }();
    const auto &reg = registry();
    const std::less<const KernelEntry *> before;
    if (!reg.empty() && !before(&e, reg.data()) && before(&e, reg.data() + reg.size())) return by_index[&e - reg.data()];
    return resources_of(e.name);  // a copy
}

}  // namespace pk
