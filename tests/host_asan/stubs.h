// What the stub launchers note while `recorded` is set.
#pragma once
#include <vector>

struct Launch {
  const char* kernel;
  int layers;
};
extern std::vector<Launch>* recorded;
