// Source text of runtime-compiled specializations (the paper's growth path,
// Sec. 3.5: a miss compiles a new specialization and installs it).
//
// A specialization is the device prelude -- the argument blocks and the very
// device bodies the precompiled kernels call (kernargs.h and
// kernels/device.h, embedded at build time) -- plus one kernel that
// overwrites the shape fields of its argument block with the key's values
// before calling the body of the planned variant. Those fields are then
// compile-time constants: loop bounds, vector counts, head strides and the
// RoPE variant branches fold, while tokens, pointers, strides and epsilons
// stay run-time arguments exactly as in the precompiled kernel.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

#include <atomic>
#include <chrono>

#include "internal.h"

namespace tri {

extern const char kJitPrelude[];      // generated by the build
extern const uint64_t kJitPreludeLen;

namespace {

const char *tf(bool b) { return b ? "true" : "false"; }

// "a.H = ...;" etc. for an argument block reached through `pre` ("a." or
// "a.rn." ...).
int shape_rn(char *o, size_t n, const char *pre, const Key &k) {
  return snprintf(o, n, "  %sH = %u;\n", pre, key_H(k));
}

int shape_rope(char *o, size_t n, const char *pre, const Key &k, const Plan &p) {
  return snprintf(o, n, "  %shd = %u; %srd = %u; %snq = %u; %snk = %u; %smode = %uu;\n", pre,
                  key_hd(k), pre, key_rd(k), pre, key_nq(k), pre, key_nk(k), pre,
                  key_rope_bits(k) | rope_geometry_bits(p.rope_slices, p.rope_tokens));
}

int shape_sw(char *o, size_t n, const char *pre, const Key &k) {
  return snprintf(o, n, "  %sI = %u;\n", pre, key_I(k));
}

// The kernel for one launch: argument type, shape fields, body call.
int kernel_text(const Key &k, const Plan &p, int i, char *o, size_t n) {
  const int32_t v = p.kvariant[i], sub = p.ksub[i];
  const unsigned dt = key_dtype(k);
  char body[160];
  char shape[200];
  const char *type = nullptr;
  if (v == RN_SPLIT) {
    type = "RnSplitArgs";
    shape_rn(shape, sizeof shape, "a.rn.", k);
    snprintf(body, sizeof body, "body_rn_split<%u, %s>(a)", dt, tf(sub != 0));
  } else if (v >= RN_SCALAR && v <= RN_WIDE) {
    type = "RnArgs";
    shape_rn(shape, sizeof shape, "a.", k);
    const char *res = tf(sub != 0);
    if (v == RN_SCALAR)
      snprintf(body, sizeof body, "body_rn_scalar<%u, %s>(a)", dt, res);
    else if (v == RN_LOOP)
      snprintf(body, sizeof body, "body_rn_loop<%u, %s>(a)", dt, res);
    else if (v == RN_WIDE)
      snprintf(body, sizeof body, "body_rn_wide<%u, %s>(a)", dt, res);
    else if (v <= RN_WAVE_2)
      snprintf(body, sizeof body, "body_rn_wave<%u, %d, %s>(a)", dt, 1 << (v - RN_WAVE_1), res);
    else
      snprintf(body, sizeof body, "body_rn_block<%u, %d, %s>(a)", dt, 1 << (v - RN_BLOCK_1), res);
  } else if (v >= ROPE_SCALAR && v <= ROPE_QKN_VEC_I) {
    type = "RopeArgs";
    shape_rope(shape, sizeof shape, "a.", k, p);
    const bool qkn = v == ROPE_QKN_SCALAR || v == ROPE_QKN_VEC || v == ROPE_QKN_VEC_I;
    const bool inter = v == ROPE_VEC_I || v == ROPE_QKN_VEC_I;
    if (v == ROPE_SCALAR || v == ROPE_QKN_SCALAR)
      snprintf(body, sizeof body, "body_rope_scalar<%u, %s>(a)", dt, tf(qkn));
    else
      snprintf(body, sizeof body, "body_rope_vec<%u, %s, %s>(a)", dt, tf(qkn), tf(inter));
  } else if (v >= SW_SCALAR && v <= SW_ROWS) {
    type = "SwArgs";
    shape_sw(shape, sizeof shape, "a.", k);
    switch (v) {
      case SW_SCALAR: snprintf(body, sizeof body, "body_sw_scalar<%u>(a)", dt); break;
      case SW_ROWS: snprintf(body, sizeof body, "body_sw_rows<%u>(a)", dt); break;
      case SW_FLAT: snprintf(body, sizeof body, "body_sw_flat<%u, 1, false>(a)", dt); break;
      case SW_FLAT_NT: snprintf(body, sizeof body, "body_sw_flat<%u, 1, true>(a)", dt); break;
    }
  } else if (v >= ELT_SCALAR && v <= ELT_ROWS) {
    type = "EltArgs";
    snprintf(shape, sizeof shape, "  a.W = %u;\n", key_H(k));
    if (v == ELT_SCALAR)
      snprintf(body, sizeof body, "body_elt_scalar<%u, %d>(a)", dt, sub);
    else if (v == ELT_ROWS)
      snprintf(body, sizeof body, "body_elt_rows<%u, %d>(a)", dt, sub);
    else
      snprintf(body, sizeof body, "body_elt_flat<%u, %d, %d>(a)", dt, sub, v == ELT_FLAT_U2 ? 2 : 1);
  } else if (v == EMB_SCALAR || v == EMB_VEC) {
    type = "EmbArgs";
    snprintf(shape, sizeof shape, "  a.H = %u; a.ids64 = %d;\n", key_H(k), sub);
    snprintf(body, sizeof body, "body_emb<%u, %s>(a)", dt, tf(v == EMB_VEC));
  } else if (v == CH_FUSED) {
    type = "ChainArgs";
    int m = shape_rn(shape, sizeof shape, "a.rn.", k);
    m += shape_rope(shape + m, sizeof shape - size_t(m), "a.rope.", k, p);
    shape_sw(shape + m, sizeof shape - size_t(m), "a.sw.", k);
    const int rn = RN_WAVE_1 + (sub >> 3);
    const bool wave = rn <= RN_WAVE_2;
    const int nv = wave ? 1 << (rn - RN_WAVE_1) : 1 << (rn - RN_BLOCK_1);
    snprintf(body, sizeof body, "body_chain<%u, %s, %d, %s, %s, %s>(a, gridDim.x)", dt, tf(wave), nv,
             tf(sub & 1), tf((sub >> 1) & 1), tf((sub >> 2) & 1));
  } else {
    return -1;
  }
  return snprintf(o, n,
                  "\nextern \"C\" __global__ __launch_bounds__(%u) void "
                  "tri_jit_kernel(tri::%s a) {\n%s  tri::dev::%s;\n}\n",
                  role_block(v, dt, key_H(k)), type, shape, body);
}

}  // namespace

char *jit_source(const Key &k, const Plan &p, int i, uint64_t *len) {
  char kernel[1024];
  const int m = kernel_text(k, p, i, kernel, sizeof kernel);
  if (m < 0 || m >= int(sizeof kernel)) return nullptr;
  const uint64_t total = kJitPreludeLen + uint64_t(m);
  char *out = static_cast<char *>(malloc(total + 1));
  if (!out) return nullptr;
  memcpy(out, kJitPrelude, kJitPreludeLen);
  memcpy(out + kJitPreludeLen, kernel, size_t(m));
  out[total] = '\0';
  *len = total;
  return out;
}

namespace {

// Everything a code object depends on besides its source text.
constexpr char kCodeFlavour[] = "gfx950 -O3 -std=c++17 -ffp-contract=off -packed-fp32-ops";

}  // namespace

uint64_t fnv1a64(const void *p, uint64_t n, uint64_t h) {
  const unsigned char *b = static_cast<const unsigned char *>(p);
  for (uint64_t i = 0; i < n; ++i) {
    h ^= b[i];
    h *= 0x100000001b3ull;
  }
  return h;
}

bool read_file(const char *path, void **data, uint64_t *n) {
  FILE *f = fopen(path, "rb");
  if (!f) return false;
  bool ok = false;
  if (fseek(f, 0, SEEK_END) == 0) {
    const long size = ftell(f);
    if (size > 0 && fseek(f, 0, SEEK_SET) == 0) {
      void *buf = malloc(size_t(size));
      if (buf && fread(buf, 1, size_t(size), f) == size_t(size)) {
        *data = buf;
        *n = uint64_t(size);
        ok = true;
      } else {
        free(buf);
      }
    }
  }
  fclose(f);
  return ok;
}

// Written under a temporary name unique to this write (process id and a
// per-process counter, so writers in other processes or threads never share
// it) and renamed, so a concurrent reader sees either no file or a whole
// one. Failures are ignored (the cache is an optimisation).
void write_file(const char *path, const void *data, uint64_t n) {
  static std::atomic<uint64_t> serial{0};
  char tmp[1100];
  if (snprintf(tmp, sizeof tmp, "%s.%ld.%llu.tmp", path, long(getpid()),
               (unsigned long long)serial.fetch_add(1, std::memory_order_relaxed)) >=
      int(sizeof tmp))
    return;
  FILE *f = fopen(tmp, "wb");
  if (!f) return;
  const bool ok = fwrite(data, 1, size_t(n), f) == size_t(n);
  if (fclose(f) != 0 || !ok || rename(tmp, path) != 0) remove(tmp);
}

int jit_build(const tri_cache *c, const char *src, uint64_t len, void **fn, void **module,
              float *ms, bool *from_dir) {
  const auto t0 = std::chrono::steady_clock::now();
  auto done = [&]() {
    *ms = float(
        std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count());
  };
  *from_dir = false;
  char path[1100] = {0};
  if (c->code_dir[0]) {
    const uint64_t h = fnv1a64(src, len, fnv1a64(kCodeFlavour, sizeof kCodeFlavour, 0xcbf29ce484222325ull));
    snprintf(path, sizeof path, "%s/tri-%016llx.co", c->code_dir, (unsigned long long)h);
    void *code = nullptr;
    uint64_t n = 0;
    if (read_file(path, &code, &n)) {
      const int st = be_load_code(code, n, fn, module);
      free(code);
      if (st == 0) {
        *from_dir = true;
        done();
        return 0;
      }
    }
  }
  void *code = nullptr;
  uint64_t n = 0;
  int st = be_compile(src, len, &code, &n);
  if (st != 0) return st;
  if (path[0]) write_file(path, code, n);
  st = be_load_code(code, n, fn, module);
  free(code);
  done();
  return st;
}

}  // namespace tri
