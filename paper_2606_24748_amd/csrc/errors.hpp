// Errors inside the library and at the C ABI.
#pragma once

#include <hip/hip_runtime_api.h>

#include <new>
#include <string>

#include "../../include/blkamg.h"

namespace blk {

// ---------------------------------------------------------------------------
// Errors: internal code throws Error; every exported function catches at the
// boundary, records the message and returns the status code.
// ---------------------------------------------------------------------------
struct Error {
  int code;
  std::string msg;
};

[[noreturn]] inline void fail(int code, const std::string& msg) { throw Error{code, msg}; }

void set_last_error(const std::string& msg);

#define BLK_REQUIRE(cond, code, msg)                      \
  do {                                                    \
    if (!(cond)) ::blk::fail((code), std::string(msg));   \
  } while (0)

#define HIP_CHECK(expr)                                                                  \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess)                                                                \
      ::blk::fail(e_ == hipErrorOutOfMemory ? BLKAMG_ENOMEM : BLKAMG_EHIP,               \
                  std::string(#expr) + ": " + hipGetErrorString(e_));                     \
  } while (0)

// Wrap the body of an exported function.
#define BLK_API_BEGIN try {
#define BLK_API_END                                              \
  return BLKAMG_OK;                                              \
  }                                                              \
  catch (const ::blk::Error& e) {                                \
    ::blk::set_last_error(e.msg);                                \
    return e.code;                                               \
  }                                                              \
  catch (const std::bad_alloc&) {                                \
    ::blk::set_last_error("host allocation failed");             \
    return BLKAMG_ENOMEM;                                        \
  }                                                              \
  catch (...) {                                                  \
    ::blk::set_last_error("unexpected internal error");          \
    return BLKAMG_EINVAL;                                        \
  }

}  // namespace blk
