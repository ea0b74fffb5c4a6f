// z-chunk depths per (kernel family, field, precision, node dims), filled by
// hts_autotune and optionally kept in the JSON file named by HTS_TUNE_CACHE.  Host code
// without HIP.  Every operator apply looks its depth up here, and calls on different
// meshes may run in several threads, one of them tuning: all access is locked.
#pragma once
#include <cctype>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <mutex>
#include <string>

namespace hts {

class TuneCache {
public:
    // the recorded depth, 0 = none
    int get(int family, int field, int prec, int NX, int NY, int NZ)
    {
        std::lock_guard<std::mutex> lk(mu);
        load();
        auto it = depth.find(key(family, field, prec, NX, NY, NZ));
        return it == depth.end() ? 0 : it->second;
    }
    void set(int family, int field, int prec, int NX, int NY, int NZ, int zc)
    {
        std::lock_guard<std::mutex> lk(mu);
        load();
        depth[key(family, field, prec, NX, NY, NZ)] = zc;
    }
    void save()
    {
        std::lock_guard<std::mutex> lk(mu);
        const char *path = getenv("HTS_TUNE_CACHE");
        if (!path) return;
        FILE *f = fopen(path, "w");
        if (!f) return;
        fprintf(f, "{");
        bool first = true;
        for (auto &kv : depth) {
            fprintf(f, "%s\n  \"%s\": %d", first ? "" : ",", kv.first.c_str(), kv.second);
            first = false;
        }
        fprintf(f, "\n}\n");
        fclose(f);
    }

private:
    std::mutex mu;
    std::map<std::string, int> depth;
    bool loaded = false;

    static std::string key(int family, int field, int prec, int NX, int NY, int NZ)
    {
        char b[96];
        snprintf(b, sizeof(b), "q%d_f%d_%s_%dx%dx%d", family, field, prec ? "fp32" : "fp64", NX, NY, NZ);
        return b;
    }
    void load()
    {
        if (loaded) return;
        loaded = true;
        const char *path = getenv("HTS_TUNE_CACHE");
        if (!path) return;
        FILE *f = fopen(path, "r");
        if (!f) return;
        char k[96];
        int v;
        // {"q1_f0_129x129x65": 8, ...}: skip the opening brace first
        int c0 = fgetc(f);
        while (c0 != EOF && isspace(c0)) c0 = fgetc(f);
        if (c0 != '{' && c0 != EOF) ungetc(c0, f);
        while (fscanf(f, " \"%95[^\"]\" : %d", k, &v) == 2) {
            depth[k] = v;
            int c = fgetc(f);
            while (c != EOF && c != ',' && c != '}') c = fgetc(f);
            if (c == '}' || c == EOF) break;
        }
        fclose(f);
    }
};

}  // namespace hts
